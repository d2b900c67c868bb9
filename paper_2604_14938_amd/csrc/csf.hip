// Surface-tension curvature of the continuum-surface-force term (Sec. 2.4,
// momentum terms, surface tension):
//   smoothing  alpha_hat_P = sum_f alpha_hat_f A_f / sum_f A_f,
//              alpha_hat_f = alpha_P + w_f (alpha_Q - alpha_P), w_f the
//              geometric weight of Q (where the centre connection meets the
//              face plane), boundary faces alpha_P; n_smooth Jacobi sweeps;
//   normal     n = grad(alpha_hat) / (|grad(alpha_hat)| + 1e-15), plain least
//              squares over interior face neighbours (App. B);
//   raw        kappa~ = -div n by the Gauss sum with n_f = n_P + w_f (n_Q - n_P);
//   step 1     kappa* = colour-weighted mean of kappa~ over P and its face
//              neighbours, w = (1 - 2|1/2 - alpha_hat|)^8;
//   step 2     kappa = the same mean of kappa* with each neighbour's weight
//              times |n_P . s_Q|^8 (s_Q the unit centre connection);
//   force      F = sigma kappa grad(alpha), plain least squares of the sharp
//              alpha.
// Every output is exact outside the cells within n_smooth + 3 rings of the
// seed (cells with alpha other than 0 or 1, or with a face neighbour of another
// alpha): a pure cell among equal neighbours keeps alpha_hat = alpha exactly
// (sums of A_f over sums of A_f), so sweep k changes alpha_hat within ring
// k - 1, the normal is nonzero one ring beyond the last sweep's, the raw
// curvature one more, and each smoothing step one more.  One streaming pass
// fills alpha_hat = alpha and zeros everywhere; each stage then runs on its own
// rings only and, beside its arithmetic, marks the next one (the unmarked
// neighbours of the newest ring, whose ids it has loaded anyway).  A group of
// lanes per cell, one face per lane, DPP sums.  The geometric weight and the
// area of every cell-face slot depend on the mesh only and are built once, by
// the first call on a mesh.
//
// The chain is bound by the number of dependent launches and by the gathers of
// each.  194,672 Voronoi cells, n_smooth 2, force: 69 us (107 to 116 us when the
// domain was grown by five passes over all faces before the first stage, every
// stage ran on the whole domain, and the two gradients, the normalisation and
// the list were launches of their own).
#include <hip/hip_runtime.h>

#include <algorithm>

#include "lsq.h"
#include "ring_ops.h"
#include "vofpc_internal.h"
#include "wave_ops.h"

namespace vofpc {

constexpr int kCsfBlock = 256;
constexpr int kCsfMaxSmooth = 100;
constexpr double kCsfEps = 1e-15;

// geometric weight of the neighbour across face f of cell P
__device__ __forceinline__ double csf_face_weight(const DevMesh &m, int f, int P, int Q) {
  const int64_t N = m.n_cells, NF = m.n_faces;
  const double S0 = m.Sf[f], S1 = m.Sf[NF + f], S2 = m.Sf[2 * NF + f];
  const double a = S0 * (m.xf[f] - m.xc[P]) + S1 * (m.xf[NF + f] - m.xc[N + P]) + S2 * (m.xf[2 * NF + f] - m.xc[2 * N + P]);
  const double b = S0 * (m.xc[Q] - m.xc[P]) + S1 * (m.xc[N + Q] - m.xc[N + P]) + S2 * (m.xc[2 * N + Q] - m.xc[2 * N + P]);
  return a / b;
}

__device__ __forceinline__ double colour_weight(double a) {
  const double w = 1.0 - 2.0 * fabs(0.5 - a);
  const double w2 = w * w, w4 = w2 * w2;
  return w4 * w4;
}

// A stage over the cells of rings 0 .. ring.  A wavefront reads the marks of
// per_wave cells and takes those of the domain 64 / W at a time, W lanes per
// cell: f(P, has, fresh, lane), fresh where the cell is of the newest ring.
// Groups beyond the wavefront's last cell repeat one with has false and write
// nothing.  No list of the domain: the marks of a mesh are a fraction of what a
// stage gathers, the cells stay in the mesh's order (a list in the order of its
// claims doubled the time of the gathers on 1,000,000 hexahedra), and marks
// need no claims (a stage that appended the next ring to a list by
// compare-and-swap took half as long again).  Blocks go to the XCDs in turn;
// runs of kStageXcdRun blocks of one XCD are neighbours.
constexpr int kStageBlock = 256, kStageXcdRun = 16;
template <int W, class F>
__device__ __forceinline__ void csf_stage(const DevMesh &m, const int8_t *mark, int ring, int per_wave, F f) {
  constexpr int kGroups = 64 / W;
  const int wl = threadIdx.x & 63, lane = wl % W, g = wl / W;
  const int64_t i = blockIdx.x / kXcd, run = (i / kStageXcdRun) * kXcd + blockIdx.x % kXcd;
  const int64_t block = run * kStageXcdRun + i % kStageXcdRun;
  const int64_t P0 = (block * (kStageBlock / 64) + (threadIdx.x >> 6)) * per_wave;
  int mk = -1;
  if (wl < per_wave && P0 + wl < m.n_cells) mk = mark[P0 + wl];
  uint64_t todo = __ballot(mk >= 0 && mk <= ring);
  const uint64_t fresh = __ballot(mk == ring);
  while (todo) {
    int at = 0;
    bool has = false;
#pragma unroll
    for (int t = 0; t < kGroups; ++t) {
      if (todo && g >= t) {
        at = __ffsll((unsigned long long)todo) - 1;
        has = g == t;
      }
      todo &= todo - 1;
    }
    f((int)(P0 + at), has, has && ((fresh >> at) & 1), lane);
  }
}
// blocks of a stage: whole turns of the XCDs' runs
static inline unsigned csf_stage_blocks(int64_t n, int per_wave) {
  const int64_t cells = kStageBlock / 64 * per_wave, turn = kXcd * kStageXcdRun;
  return (unsigned)std::max<int64_t>(1, ((n + cells - 1) / cells + turn - 1) / turn * turn);
}
// the neighbour Q of a cell of the newest ring enters the next one
__device__ __forceinline__ void csf_grow(int8_t *mark, int Q, int ring) {
  if (mark[Q] < 0) mark[Q] = (int8_t)(ring + 1);   // (every writer writes the same)
}

// per cell-face slot, once per mesh: the geometric weight of the neighbour
// (as seen from the slot's cell) and the face area
__global__ __launch_bounds__(kCsfBlock) void csf_slot_kernel(DevMesh m, double *slot) {
  constexpr int kLanes = 16, kCells = kCsfBlock / kLanes;
  const int64_t NF = m.n_faces, NS = m.cell_face_off[m.n_cells];
  const int lane = threadIdx.x % kLanes;
  for (int64_t P = blockIdx.x * (int64_t)kCells + threadIdx.x / kLanes; P < m.n_cells;
       P += (int64_t)gridDim.x * kCells) {
    for (int64_t i = m.cell_face_off[P] + lane; i < m.cell_face_off[P + 1]; i += kLanes) {
      const int f = m.cell_face[i];
      const int Q = m.cf_nbr[i];
      const double S0 = m.Sf[f], S1 = m.Sf[NF + f], S2 = m.Sf[2 * NF + f];
      slot[i] = Q >= 0 ? csf_face_weight(m, f, (int)P, Q) : 0.0;
      slot[NS + i] = sqrt(S0 * S0 + S1 * S1 + S2 * S2);
    }
  }
}

template <int W>
__global__ __launch_bounds__(kStageBlock) void csf_smooth_kernel(DevMesh m, const double *slot, int8_t *mark,
                                                                int ring, int per_wave, const double *cur, double *nxt) {
  const int64_t NS = m.cell_face_off[m.n_cells];
  csf_stage<W>(m, mark, ring, per_wave, [&](int P, bool has, bool fresh, int lane) {
    const int64_t i0 = m.cell_face_off[P], i1 = has ? m.cell_face_off[P + 1] : i0;
    const double aP = cur[P];
    double num = 0.0, den = 0.0;
    for (int64_t i = i0 + lane; i < i1; i += W) {
      const int Q = m.cf_nbr[i];
      const double A = slot[NS + i];
      const double af = Q >= 0 ? aP + slot[i] * (cur[Q] - aP) : aP;
      num += af * A;
      den += A;
      if (Q >= 0 && fresh) csf_grow(mark, Q, ring);
    }
    num = gsum<W>(num);
    den = gsum<W>(den);
    if (has && lane == 0) nxt[P] = num / den;
  });
}

// every cell: alpha_hat = alpha (both smoothing buffers) and every other
// output 0, their values outside the domain; cells with alpha other than 0
// or 1 are marked for ring 0
__global__ __launch_bounds__(kCsfBlock) void csf_fill_kernel(int64_t N, const double *alpha, double *ah, double *tmp,
                                                             double *n, double *kr, double *ks, double *kappa,
                                                             double *F, int8_t *mark) {
  for (int64_t P = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; P < N; P += (int64_t)gridDim.x * blockDim.x) {
    const double a = alpha[P];
    mark[P] = (a == 0.0 || a == 1.0) ? -1 : 0;
    ah[P] = a;
    tmp[P] = a;
    n[P] = 0.0;
    n[N + P] = 0.0;
    n[2 * N + P] = 0.0;
    kr[P] = 0.0;
    ks[P] = 0.0;
    kappa[P] = 0.0;
    if (F) {
      F[P] = 0.0;
      F[N + P] = 0.0;
      F[2 * N + P] = 0.0;
    }
  }
}

// ring 0, the rest of it: cells with a face neighbour of another alpha
__global__ __launch_bounds__(kRingBlock) void csf_seed_faces_kernel(DevMesh m, const double *alpha, int8_t *mark) {
  const int64_t f0 = (blockIdx.x * (int64_t)kRingBlock + threadIdx.x) * kRingRun;
  if (f0 >= m.n_faces) return;
  int o[kRingRun], q[kRingRun];
  ring_faces(m, f0, o, q);
  double ao[kRingRun], aq[kRingRun];
#pragma unroll
  for (int t = 0; t < kRingRun; ++t) {
    ao[t] = alpha[o[t]];
    aq[t] = q[t] >= 0 ? alpha[q[t]] : ao[t];
  }
#pragma unroll
  for (int t = 0; t < kRingRun; ++t)
    if (q[t] >= 0 && ao[t] != aq[t]) {
      mark[o[t]] = 0;
      mark[q[t]] = 0;
    }
}

// The normal from the plain gradient of alpha_hat over interior neighbours, and
// the plain gradient of alpha into F where the force is asked for: one stencil
// matrix and one walk for both.
template <int W, bool FORCE>
__global__ __launch_bounds__(kStageBlock) void csf_normal_kernel(DevMesh m, int8_t *mark, int ring, int per_wave,
                                                                const double *alpha, const double *ah, double *n,
                                                                double *F) {
  const int64_t N = m.n_cells;
  csf_stage<W>(m, mark, ring, per_wave, [&](int P, bool has, bool fresh, int lane) {
    const int64_t i0 = m.cell_face_off[P], i1 = has ? m.cell_face_off[P + 1] : i0;
    const double4 xP = m.xr[P];
    const double hP = ah[P], aP = FORCE ? alpha[P] : 0.0;
    LsqSums L;
    double c0 = 0.0, c1 = 0.0, c2 = 0.0;
    for (int64_t i = i0 + lane; i < i1; i += W) {
      const int Q = m.cf_nbr[i];
      if (Q < 0) continue;
      const double4 xQ = m.xr[Q];
      const double r0 = xQ.x - xP.x, r1 = xQ.y - xP.y, r2 = xQ.z - xP.z;
      L.add(r0, r1, r2, ah[Q] - hP, 0);
      if (FORCE) {
        const double da = alpha[Q] - aP;
        c0 += r0 * da; c1 += r1 * da; c2 += r2 * da;
      }
      if (fresh) csf_grow(mark, Q, ring);
    }
    lsq_reduce<W>(L);
    double g0, g1, g2;
    (void)lsq_solve(L, g0, g1, g2);   // a singular stencil gives zero
    const double len = sqrt(g0 * g0 + g1 * g1 + g2 * g2) + kCsfEps;
    if (has && lane < 3) n[lane * N + P] = (lane == 0 ? g0 : lane == 1 ? g1 : g2) / len;
    if (FORCE) {
      L.b0 = gsum<W>(c0);
      L.b1 = gsum<W>(c1);
      L.b2 = gsum<W>(c2);
      (void)lsq_solve(L, g0, g1, g2);
      if (has && lane < 3) F[lane * N + P] = lane == 0 ? g0 : lane == 1 ? g1 : g2;
    }
  });
}

template <int W>
__global__ __launch_bounds__(kStageBlock) void csf_divergence_kernel(DevMesh m, const double *slot, int8_t *mark,
                                                                    int ring, int per_wave, const double *n, double *kraw) {
  const int64_t N = m.n_cells;
  csf_stage<W>(m, mark, ring, per_wave, [&](int P, bool has, bool fresh, int lane) {
    const int64_t i0 = m.cell_face_off[P], i1 = has ? m.cell_face_off[P + 1] : i0;
    const double p0 = n[P], p1 = n[N + P], p2 = n[2 * N + P];
    double div = 0.0;
    for (int64_t i = i0 + lane; i < i1; i += W) {
      const int Q = m.cf_nbr[i];
      const double *S = m.cf_S + 3 * i;
      double f0 = p0, f1 = p1, f2 = p2;
      if (Q >= 0) {
        const double w = slot[i];
        f0 = p0 + w * (n[Q] - p0);
        f1 = p1 + w * (n[N + Q] - p1);
        f2 = p2 + w * (n[2 * N + Q] - p2);
        if (fresh) csf_grow(mark, Q, ring);
      }
      div += f0 * S[0] + f1 * S[1] + f2 * S[2];
    }
    div = gsum<W>(div);
    if (has && lane == 0) kraw[P] = -div / m.V[P];
  });
}

template <int W>
__global__ __launch_bounds__(kStageBlock) void csf_step1_kernel(DevMesh m, int8_t *mark, int ring, int per_wave, const double *ah,
                                                               const double *kraw, double *kstar) {
  csf_stage<W>(m, mark, ring, per_wave, [&](int P, bool has, bool fresh, int lane) {
    const int64_t i0 = m.cell_face_off[P], i1 = has ? m.cell_face_off[P + 1] : i0;
    double num = 0.0, den = 0.0;
    for (int64_t i = i0 + lane; i < i1; i += W) {
      const int Q = m.cf_nbr[i];
      if (Q < 0) continue;
      const double wQ = colour_weight(ah[Q]);
      num += kraw[Q] * wQ;
      den += wQ;
      if (fresh) csf_grow(mark, Q, ring);
    }
    num = gsum<W>(num);
    den = gsum<W>(den);
    if (has && lane == 0) {
      const double wP = colour_weight(ah[P]);
      kstar[P] = (kraw[P] * wP + num) / (wP + den + kCsfEps);
    }
  });
}

// step 2, and the force where asked: F holds grad(alpha) on entry
template <int W>
__global__ __launch_bounds__(kStageBlock) void csf_step2_kernel(DevMesh m, int8_t *mark, int ring, int per_wave, const double *ah,
                                                               const double *n, const double *kstar, double *kappa,
                                                               double sigma, double *F) {
  const int64_t N = m.n_cells;
  csf_stage<W>(m, mark, ring, per_wave, [&](int P, bool has, bool fresh, int lane) {
    const int64_t i0 = m.cell_face_off[P], i1 = has ? m.cell_face_off[P + 1] : i0;
    const double n0 = n[P], n1 = n[N + P], n2 = n[2 * N + P];
    const double4 xP = m.xr[P];
    double num = 0.0, den = 0.0;
    for (int64_t i = i0 + lane; i < i1; i += W) {
      const int Q = m.cf_nbr[i];
      if (Q < 0) continue;
      const double4 xQ = m.xr[Q];
      const double s0 = xQ.x - xP.x, s1 = xQ.y - xP.y, s2 = xQ.z - xP.z;
      const double len = sqrt(s0 * s0 + s1 * s1 + s2 * s2);
      const double c = fabs((n0 * s0 + n1 * s1 + n2 * s2) / len);
      const double c2 = c * c, c4 = c2 * c2;
      const double w = colour_weight(ah[Q]) * (c4 * c4);
      num += kstar[Q] * w;
      den += w;
    }
    num = gsum<W>(num);
    den = gsum<W>(den);
    const double wP = colour_weight(ah[P]);
    const double k = (kstar[P] * wP + num) / (wP + den + kCsfEps);
    if (has && lane == 0) kappa[P] = k;
    if (F && has && lane < 3) F[lane * N + P] *= sigma * k;
  });
}

template <int W>
static void csf_chain(vofpc_ctx ctx, vofpc_mesh M, const double *alpha, int n_smooth, double sigma, double *alpha_hat,
                      double *n, double *kr, double *kappa, double *force) {
  const int64_t N = M->d.n_cells;
  hipStream_t s = ctx->stream;
  double *tmp = M->csf_buf;            // smoothing ping-pong
  double *ks = M->csf_buf + 2 * N;     // step-1 curvature
  int8_t *mark = M->csf_mark;
  // one turn of a wavefront's groups, so that no wavefront runs several in a
  // row; more where the blocks would pass 48 per CU, whose launch then costs more
  // than a second turn (us with 4 / 8 / 16 / 32 cells: 194,672 Voronoi cells
  // 69 / 71 / 87 / 90, 410,758: 242 / 228 / 229 / 252; 125,000 hexahedra
  // 79 / 63 / 66 / 79, 1,000,000: 445 / 298 / 267 / 248)
  int per_wave = 64 / W;
  while (per_wave < 64 && N > (int64_t)ctx->n_cu * 48 * (kStageBlock / 64) * per_wave) per_wave *= 2;
  const unsigned gC = csf_stage_blocks(N, per_wave);
  const unsigned gE = (unsigned)std::max<int64_t>(1, std::min<int64_t>((N + kCsfBlock - 1) / kCsfBlock,
                                                                       (int64_t)ctx->n_cu * 8));
  csf_fill_kernel<<<gE, kCsfBlock, 0, s>>>(N, alpha, alpha_hat, tmp, n, kr, ks, kappa, force, mark);
  csf_seed_faces_kernel<<<ring_face_blocks(M->d.n_faces), kRingBlock, 0, s>>>(M->d, alpha, mark);
  // smoothing: sweep k writes alpha_hat when n_smooth - 1 - k is even, so the
  // last sweep lands there
  const double *src = alpha;
  for (int k = 0; k < n_smooth; ++k) {
    double *dst = ((n_smooth - 1 - k) % 2 == 0) ? alpha_hat : tmp;
    csf_smooth_kernel<W><<<gC, kStageBlock, 0, s>>>(M->d, M->csf_slot, mark, k, per_wave, src, dst);
    src = dst;
  }
  const int r = n_smooth;
  if (force) csf_normal_kernel<W, true><<<gC, kStageBlock, 0, s>>>(M->d, mark, r, per_wave, alpha, alpha_hat, n, force);
  else csf_normal_kernel<W, false><<<gC, kStageBlock, 0, s>>>(M->d, mark, r, per_wave, alpha, alpha_hat, n, nullptr);
  csf_divergence_kernel<W><<<gC, kStageBlock, 0, s>>>(M->d, M->csf_slot, mark, r + 1, per_wave, n, kr);
  csf_step1_kernel<W><<<gC, kStageBlock, 0, s>>>(M->d, mark, r + 2, per_wave, alpha_hat, kr, ks);
  csf_step2_kernel<W><<<gC, kStageBlock, 0, s>>>(M->d, mark, r + 3, per_wave, alpha_hat, n, ks, kappa, sigma, force);
}

}  // namespace vofpc

using namespace vofpc;

extern "C" vofpc_status vofpc_csf_opts_default(vofpc_csf_opts *o) {
  clear_error();
  VOFPC_REQUIRE(o, VOFPC_E_INVALID_ARG, "csf_opts_default: null argument");
  o->n_smooth = 2;
  o->sigma = 1.0;
  return VOFPC_OK;
}

extern "C" vofpc_status vofpc_curvature(vofpc_ctx ctx, vofpc_mesh M, const double *alpha, const vofpc_csf_opts *opts,
                                        double *alpha_hat, double *n, double *kappa_raw, double *kappa,
                                        double *force) {
  clear_error();
  VOFPC_REQUIRE(ctx && M && alpha && alpha_hat && n && kappa, VOFPC_E_INVALID_ARG, "curvature: null argument");
  VOFPC_REQUIRE(M->ctx && M->ctx->device == ctx->device, VOFPC_E_STATE, "curvature: mesh on another device");
  vofpc_csf_opts o;
  if (opts) o = *opts; else vofpc_csf_opts_default(&o);
  VOFPC_REQUIRE(o.n_smooth >= 0 && o.n_smooth <= kCsfMaxSmooth, VOFPC_E_INVALID_ARG, "curvature: n_smooth out of range");
  VOFPC_HIP(hipSetDevice(ctx->device));
  const int64_t N = M->d.n_cells;
  hipStream_t s = ctx->stream;
  if (!M->csf_buf) {
    hipStreamCaptureStatus cs = hipStreamCaptureStatusNone;
    VOFPC_HIP(hipStreamIsCapturing(s, &cs));
    VOFPC_REQUIRE(cs == hipStreamCaptureStatusNone, VOFPC_E_STATE,
                  "curvature: the first call on a mesh sets up its buffers and must not be captured");
    void *a = nullptr, *b = nullptr;
    vofpc_status st;
    if ((st = mesh_scratch_alloc(M, 24 * (size_t)N, &a)) || (st = mesh_scratch_alloc(M, (size_t)N, &b)))
      return st;
    M->csf_buf = (double *)a;
    M->csf_mark = (int8_t *)b;
  }
  if (!M->csf_slot) {
    // per-slot weights and areas: fixed by the geometry, built once
    hipStreamCaptureStatus cs = hipStreamCaptureStatusNone;
    VOFPC_HIP(hipStreamIsCapturing(s, &cs));
    VOFPC_REQUIRE(cs == hipStreamCaptureStatusNone, VOFPC_E_STATE,
                  "curvature: the first call on a mesh sets up its buffers and must not be captured");
    void *a = nullptr;
    vofpc_status st = mesh_scratch_alloc(M, 16 * (size_t)std::max<int64_t>(M->ncf, 1), &a);
    if (st) return st;
    M->csf_slot = (double *)a;
    csf_slot_kernel<<<(unsigned)std::max<int64_t>(1, std::min<int64_t>((N + 15) / 16, (int64_t)ctx->n_cu * 16)),
                      kCsfBlock, 0, s>>>(M->d, M->csf_slot);
    VOFPC_HIP(hipGetLastError());
  }
  double *kr = kappa_raw ? kappa_raw : M->csf_buf + N;   // raw curvature
  // eight lanes where no cell has more faces (the same sums in the same order),
  // else one face per lane of a DPP row
  if (M->max_nf <= 8) csf_chain<8>(ctx, M, alpha, o.n_smooth, o.sigma, alpha_hat, n, kr, kappa, force);
  else csf_chain<16>(ctx, M, alpha, o.n_smooth, o.sigma, alpha_hat, n, kr, kappa, force);
  VOFPC_HIP(hipGetLastError());
  return VOFPC_OK;
}

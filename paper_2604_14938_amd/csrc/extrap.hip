// Phase gradients at the interface by pseudo-time extrapolation
// (Eq. extrapolation, Sec. 2.4.4), each gradient component separately:
//   the domain D is the mixed cells and `layers` rings of interior face
//   neighbours around them; on D, G_l = G_v = the interface-modified gradient;
//   a liquid cell (alpha >= 1/2) keeps G_l and advances G_v, a vapour cell
//   keeps G_v and advances G_l, with velocity c = sgn(alpha - 1/2) n (n: the
//   interface normal where the cell has an interface, else the unit plain
//   least-squares gradient of alpha over interior neighbours);
//   first-order upwind, Jacobi: with w_f = -c.S_f over the faces whose
//   neighbour is in D and c.S_f < 0, F_P <- F_P + theta (sum w_f F_Q / w - F_P),
//   theta = min(dtau w / V_P, 1), dtau = the smallest centre distance of two
//   face neighbours; stop at the first sweep whose largest change is below
//   tol, or after max_iter sweeps.
//
// The domain is grown, listed and given its stencil by kernels of their own;
// one persistent kernel then runs every sweep and writes the outputs.  A block
// keeps its first cells' stencils and values in registers; the iterates go
// through memory at agent scope (relaxed atomic loads and stores, which meet
// beyond the per-XCD L2 caches), so a sweep needs no cache write-back or
// invalidation, only a barrier of flags: each block posts the sweep's number
// and whether any of its cells still changes, and reads the others'.  With a
// launch per sweep all of max_iter were issued whether they had work or not:
// 500 us a call on 194,672 Voronoi cells (19 sweeps of 120, a domain of 16,000
// cells), now 149.  Five kernels of set-up, 41 us of that, stay: each needs
// the whole of the one before.
#include <hip/hip_runtime.h>

#include <algorithm>

#include "lsq.h"
#include "ring_ops.h"
#include "sweep_sync.h"
#include "vofpc_internal.h"
#include "wave_ops.h"

namespace vofpc {

constexpr int kExBlock = 256;
constexpr int8_t kExInterface = 127;    // mark of a domain cell with an interface (layers end at 100)

__device__ __forceinline__ bool is_mixed(double a, double eps) { return a > eps && a < 1.0 - eps; }

// layer 0: the mixed cells; everything else outside; the list length, the
// barrier flags and the report are reset
__global__ __launch_bounds__(kExBlock) void ex_init_kernel(int64_t n, const double *alpha, double eps, int8_t *mark,
                                                           int32_t *info, uint32_t *flag, int32_t *report) {
  const int64_t P = blockIdx.x * (int64_t)kExBlock + threadIdx.x;
  if (P < n) mark[P] = is_mixed(alpha[P], eps) ? 0 : -1;
  for (int64_t i = P; i < kSyncWords; i += (int64_t)gridDim.x * kExBlock) flag[i] = 0;
  if (P == 0) info[1] = 0;
  if (P < 2 && report) report[P] = 0;
}

// the list of the domain, by the first blocks; by the others, the mixed entry
// of every domain cell with an interface, and its mark (still at least 0, so
// the list does not care which comes first)
__global__ __launch_bounds__(kRingBlock) void ex_list_kernel(int64_t n, int8_t *mark, int32_t *list, int32_t *len,
                                                             int list_blocks, const int32_t *mixed,
                                                             const int32_t *counts, vofpc_interface itf,
                                                             int32_t *entry) {
  if ((int)blockIdx.x < list_blocks) {
    ring_list_block(n, [&](int64_t P) { return mark[P] >= 0; }, list, len, blockIdx.x);
    return;
  }
  int64_t cnt = counts[0];
  if (cnt > itf.cap) cnt = itf.cap;
  const int64_t stride = (int64_t)(gridDim.x - list_blocks) * kRingBlock;
  for (int64_t k = (int64_t)(blockIdx.x - list_blocks) * kRingBlock + threadIdx.x; k < cnt; k += stride) {
    const int P = mixed[k];
    if (!(itf.A[k] > 0) || mark[P] < 0) continue;
    mark[P] = kExInterface;
    entry[P] = (int32_t)k;
  }
}

struct ExParams {
  DevMesh m;
  const double *alpha, *T, *Tb;
  double T_sat;
  vofpc_interface itf;
  const int32_t *list, *entry;
  double *wup;      // per cell-face slot: upwind weights w_f / sum w, packed at the front of each cell's slots
  int32_t *upn;     // per cell-face slot: the neighbour of each packed upwind weight
  int2 *upr;        // per domain entry: first slot and number of its packed upwind weights
  double *theta;    // per domain entry: pseudo-time fraction min(dtau sum w / V, 1), 0 without upwind faces
  const int32_t *info;
  uint32_t *flag;
  const int8_t *mark;
  double *buf;   // [2][N][kExRec]
  double dtau, tol;
  int max_iter;
  double *gl, *gv;
  int32_t *report;
};

constexpr int kExLanes = 8;   // lanes per domain cell in the stencil (half a DPP row)
// The two iterates of both fields: one 64-byte record per cell and iterate,
// G_l in words 0-2 and G_v in words 3-5, so a neighbour's gathered
// components share one cache line.
constexpr int kExRec = 8;

// Domain entry j by a group of kExLanes lanes, fixed for the whole iteration:
//   - the interface-modified gradient of T, the start of both fields, written
//     to both iterates and to p.gl;
//   - the advection direction c = sgn(alpha - 1/2) n, n the interface normal
//     where the cell has an interface, else the unit plain gradient of alpha
//     over interior neighbours;
//   - the faces with c.S_f < 0 (S_f outward) whose neighbour is in the domain
//     get w_f = -c.S_f; those faces, in slot order, are packed at the front of
//     the cell's slot range as (w_f / sum w, neighbour), the entry keeps
//     (first slot, count) and theta = min(dtau sum w / V_P, 1) (0 when no
//     face is upwind: no update).
// Both gradients come from one walk over the faces: their stencils share the
// neighbours' centres and alphas.
__device__ __forceinline__ void ex_stencil(const ExParams &p, int64_t j, int lane) {
  const DevMesh &m = p.m;
  const int64_t N = m.n_cells, NF = m.n_faces;
  const int P = p.list[j];
  const int64_t i0 = m.cell_face_off[P], i1 = m.cell_face_off[P + 1];
  const double4 xP = m.xr[P];
  const double aP = p.alpha[P], TP = p.T[P];
  const int8_t mk = p.mark[P];
  LsqSums L, A;   // of T, of alpha
  for (int64_t i = i0 + lane; i < i1; i += kExLanes) {
    const int q = m.cf_nbr[i];
    if (q >= 0) {
      const double4 xQ = m.xr[q];
      double r0 = xQ.x - xP.x, r1 = xQ.y - xP.y, r2 = xQ.z - xP.z;
      const double aQ = p.alpha[q];
      double val = p.T[q];
      A.add(r0, r1, r2, aQ - aP, 0);
      if ((aP - 0.5) * (aQ - 0.5) < 0.0) {
        const double t = (aP - 0.5) / (aP - aQ);
        r0 *= t; r1 *= t; r2 *= t;
        val = p.T_sat;
      }
      L.add(r0, r1, r2, val - TP, 0);
    } else if (q == -1) {
      const int f = m.cell_face[i];
      L.add(m.xf[f] - xP.x, m.xf[NF + f] - xP.y, m.xf[2 * NF + f] - xP.z, p.Tb[f] - TP, 0);
    }
  }
  lsq_reduce<kExLanes>(L);
  double g[3];
  (void)lsq_solve(L, g[0], g[1], g[2]);   // a singular stencil gives zero
  double c0, c1, c2;
  if (mk == kExInterface) {
    const int64_t k = p.entry[P], cap = p.itf.cap;
    c0 = p.itf.n[k]; c1 = p.itf.n[cap + k]; c2 = p.itf.n[2 * cap + k];
  } else {
    lsq_reduce<kExLanes>(A);
    (void)lsq_solve(A, c0, c1, c2);
    const double len = sqrt(c0 * c0 + c1 * c1 + c2 * c2);
    c0 = len > 0 ? c0 / len : 0.0;
    c1 = len > 0 ? c1 / len : 0.0;
    c2 = len > 0 ? c2 / len : 0.0;
  }
  if (lane < 3) {
    const double v = lane == 0 ? g[0] : (lane == 1 ? g[1] : g[2]);
    double *rec0 = p.buf + (int64_t)P * kExRec, *rec1 = p.buf + ((int64_t)N + P) * kExRec;
    rec0[lane] = v;
    rec0[3 + lane] = v;
    rec1[lane] = v;
    rec1[3 + lane] = v;
    p.gl[lane * N + P] = v;
  }
  const double sgn = aP >= 0.5 ? 1.0 : -1.0;
  c0 *= sgn; c1 *= sgn; c2 *= sgn;
  // w_f of slot i: -c.S_f when that is positive and the neighbour Q is in the domain, else 0
  auto weight = [&](int64_t i, int &Q) -> double {
    Q = m.cf_nbr[i];
    if (Q < 0 || p.mark[Q] < 0) return 0.0;
    const double *S = m.cf_S + 3 * i;
    const double cs = c0 * S[0] + c1 * S[1] + c2 * S[2];
    return cs < 0.0 ? -cs : 0.0;
  };
  double w = 0.0;
  for (int64_t i = i0 + lane; i < i1; i += kExLanes) {
    int Q;
    w += weight(i, Q);
  }
  w = gsum<kExLanes>(w);
  // the lanes of a group share the cell, so they run the same rounds; each
  // round packs its upwind slots after those of the rounds before
  const int first = (threadIdx.x & 63) & ~(kExLanes - 1);
  const uint64_t below = (1ull << lane) - 1;
  int n = 0;
  for (int64_t k0 = i0; k0 < i1; k0 += kExLanes) {
    const int64_t i = k0 + lane;
    int Q = -1;
    const double wf = (i < i1 && w > 0.0) ? weight(i, Q) : 0.0;
    const bool up = wf > 0.0;
    const uint64_t gm = (__ballot(up) >> first) & ((1ull << kExLanes) - 1);
    if (up) {
      const int64_t o = i0 + n + __popcll(gm & below);
      p.wup[o] = wf / w;
      p.upn[o] = Q;
    }
    n += __popcll(gm);
  }
  if (lane == 0) {
    double th = 0.0;
    if (w > 0.0) {
      th = p.dtau * w / m.V[P];
      if (th > 1.0) th = 1.0;
    }
    p.theta[j] = th;
    p.upr[j] = make_int2((int)i0, n);
  }
}

__global__ __launch_bounds__(kExBlock) void ex_stencil_kernel(ExParams p) {
  constexpr int kCells = kExBlock / kExLanes;
  const int64_t nd = p.info[1];
  const int lane = threadIdx.x % kExLanes;
  for (int64_t j = blockIdx.x * (int64_t)kCells + threadIdx.x / kExLanes; j < nd; j += (int64_t)gridDim.x * kCells)
    ex_stencil(p, j, lane);
}

// Values that blocks exchange within the sweep kernel: agent scope, relaxed.
__device__ __forceinline__ double agent_load(const double *a) {
  return __hip_atomic_load(a, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void agent_store(double *a, double v) {
  __hip_atomic_store(a, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// The lanes of a wavefront and its agent-scope accesses for the flags.
struct WaveSync {
  static constexpr int kLanes = 64;
  __device__ __forceinline__ int lane() const { return threadIdx.x & 63; }
  __device__ __forceinline__ uint32_t load(const uint32_t *a) const {
    return __hip_atomic_load(a, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
  __device__ __forceinline__ void store(uint32_t *a, uint32_t v) const {
    __hip_atomic_store(a, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
  __device__ __forceinline__ uint32_t fetch_add(uint32_t *a, uint32_t v) const {
    return __hip_atomic_fetch_add(a, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
  __device__ __forceinline__ uint32_t fetch_or(uint32_t *a, uint32_t v) const {
    return __hip_atomic_fetch_or(a, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
  __device__ __forceinline__ bool any(bool b) const { return __any(b); }
  __device__ __forceinline__ int first(int v) const { return __builtin_amdgcn_readfirstlane(v); }
};

// The blocks that take part in the sweeps (sweep_sync.h), of an ordinary launch:
// a cooperative one promises residency for 20 to 30 us more, and 200 us when
// several processes share the device.  This block's number, or -1; the sweeps
// done before it takes part and the number of blocks then.
__device__ __forceinline__ int sweep_enter(uint32_t *flag, int want, int &sweeps, int &nb) {
  __shared__ int in[3];
  if (threadIdx.x < 64) {
    int e, n;
    const int id = sync_enter(WaveSync(), flag, want, e, n);
    if (threadIdx.x == 0) {
      in[0] = id;
      in[1] = e;
      in[2] = n;
    }
  }
  __syncthreads();
  sweeps = in[1];
  nb = in[2];
  return in[0];
}

// Barrier over the nb blocks that take part (this one number id), epoch 1, 2,
// ...: every agent-scope store made before it is seen by every agent-scope load
// after it.  Returns in `any` whether some block brought `mine`, and in `next`
// the number of blocks of the next sweep.  The first wavefront polls for its
// block (1.6 us a barrier of 16 blocks, 2.4 of 64, 3.2 of 256; with every
// wavefront in the poll 4.3 and 6.2).  All blocks run, so the wait ends; should a
// flag never come, it ends with false (kSyncWaitPolls).
__device__ __forceinline__ bool sweep_barrier(uint32_t *flag, int id, int nb, int want, uint32_t epoch, bool mine,
                                              bool &any, int &next) {
  __shared__ int seen[2];   // bit 0: some block brought mine, bit 1: a wait ended without its flag; the next blocks
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");   // this wavefront's stores have reached the agent's memory
  const int b = __syncthreads_or(mine ? 1 : 0);
  if (threadIdx.x < 64) {
    bool some;
    const bool ok = sync_barrier(WaveSync(), flag, id, nb, want, epoch, b != 0, some);
    if (threadIdx.x == 0) {
      seen[0] = (some ? 1 : 0) | (ok ? 0 : 2);
      seen[1] = nb;
    }
  }
  __syncthreads();
  const int r = seen[0];   // the next write to it comes after the next barrier's __syncthreads_or
  next = seen[1];
  any = (r & 1) != 0;
  return (r & 2) == 0;
}

// Every Jacobi sweep, and the outputs.  Four lanes per domain cell, one for
// each component of the advanced field (the last one only keeps the groups
// aligned): the three lanes of a cell read a neighbour's components as one
// 24-byte piece of its record, so a sweep makes one request per upwind slot.
// A group's first cell stays in registers (its value, and up to kItSlots
// weights and neighbours); its further cells (domains beyond 65,536 cells) are
// read again each sweep (two kept cells spill: 8.1 us a sweep of 16,000 cells
// for 5.7).  The kept field was written to both iterates at the
// start and is not touched.  After a sweep whose largest change is below tol,
// or max_iter sweeps, the newest values go to the outputs.  Only as many blocks
// as the domain fills take part: a sweep over 16,000 cells is bound by the
// round trips of the gathers and of its barrier.  A block's first cells depend
// on its number alone; its further cells on how many blocks sweep, which grows
// when blocks come late, so those are read from memory at every sweep.
constexpr int kItBlock = 1024, kItLanes = 4, kItCells = kItBlock / kItLanes, kItSlots = 10;
__global__ __launch_bounds__(kItBlock) void ex_iterate_kernel(ExParams p) {
  const int64_t N = p.m.n_cells, nd = p.info[1];
  const int want = (int)std::min<int64_t>(gridDim.x, std::max<int64_t>(1, (nd + kItCells - 1) / kItCells));
  int id = (int)blockIdx.x, nb = want, sweeps = 0;
  if (id >= want) return;
  if (p.max_iter > 1) {   // (a single sweep has no barrier)
    id = sweep_enter(p.flag, want, sweeps, nb);
    if (id < 0) return;
  }
  const int d = threadIdx.x % kItLanes;
  const bool comp = d < 3;
  const int64_t j0 = (int64_t)id * kItCells + threadIdx.x / kItLanes;
  int64_t stride = (int64_t)nb * kItCells;
  // the group's first cell: word `at` of its record (its advanced component
  // d) with its value, and the neighbours and weights of its first slots
  int P = 0, at = 0, cnt = 0, first = 0, nbr[kItSlots];
  double th = 0.0, v = 0.0, w[kItSlots];
  const bool has = comp && j0 < nd;
  if (has) {
    P = p.list[j0];
    at = (p.alpha[P] >= 0.5 ? 3 : 0) + d;   // G_v advances in liquid, G_l in vapour
    const int2 ur = p.upr[j0];
    first = ur.x;
    cnt = ur.y;
    th = p.theta[j0];
    v = agent_load(p.buf + (int64_t)(sweeps & 1) * kExRec * N + (int64_t)P * kExRec + at);
  }
#pragma unroll
  for (int k = 0; k < kItSlots; ++k) {
    w[k] = k < cnt ? p.wup[first + k] : 0.0;
    nbr[k] = k < cnt ? p.upn[first + k] : 0;
  }
  int in = nb;   // blocks let in, as the leader knows it
  bool ok = true;
  while (sweeps < p.max_iter) {
    const double *cur = p.buf + (int64_t)(sweeps & 1) * kExRec * N;
    double *nxt = p.buf + (int64_t)((sweeps + 1) & 1) * kExRec * N;
    double change = 0.0;
    if (has) {
      const double *from = cur + at;
      double q[kItSlots], a = 0.0;
#pragma unroll
      for (int k = 0; k < kItSlots; ++k) q[k] = k < cnt ? agent_load(from + (int64_t)nbr[k] * kExRec) : 0.0;
#pragma unroll
      for (int k = 0; k < kItSlots; ++k) a += w[k] * q[k];
      for (int k = kItSlots; k < cnt; ++k)
        a += p.wup[first + k] * agent_load(from + (int64_t)p.upn[first + k] * kExRec);
      const double n = v + th * (a - v);
      change = fmax(change, fabs(n - v));   // (a NaN does not hold the others back)
      v = n;
      agent_store(nxt + (int64_t)P * kExRec + at, n);
    }
    for (int64_t j = j0 + stride; comp && j < nd; j += stride) {
      const int C = p.list[j], c = (p.alpha[C] >= 0.5 ? 3 : 0) + d;
      const int2 ur = p.upr[j];
      const double o = agent_load(cur + (int64_t)C * kExRec + c), t = p.theta[j];
      double a = 0.0;
#pragma unroll 8
      for (int k = 0; k < ur.y; ++k)
        a += p.wup[ur.x + k] * agent_load(cur + (int64_t)p.upn[ur.x + k] * kExRec + c);
      const double n = o + t * (a - o);
      change = fmax(change, fabs(n - o));
      agent_store(nxt + (int64_t)C * kExRec + c, n);
    }
    ++sweeps;
    if (sweeps == p.max_iter) break;   // (each group reads back its own cells alone)
    bool more;
    ok = sweep_barrier(p.flag, id, nb, want, (uint32_t)sweeps, !(change < p.tol), more, in);
    if (!ok || !more) break;
    nb = in;
    stride = (int64_t)nb * kItCells;
  }
  if (id == 0 && in < want && threadIdx.x < 64) sync_close(WaveSync(), p.flag, in);
  // outputs: the advanced field from the newest iterate, the kept one from the
  // gradient both started from (in gl)
  const double *fin = p.buf + (int64_t)(sweeps & 1) * kExRec * N;
  auto put = [&](int C, int c, double x) {
    const int64_t o = d * N + C;
    if (!ok) x = __builtin_nan("");   // no result rather than an early one
    if (c >= 3) {
      p.gv[o] = x;
    } else {
      p.gv[o] = p.gl[o];
      p.gl[o] = x;
    }
  };
  if (has) put(P, at, v);
  for (int64_t j = j0 + stride; comp && j < nd; j += stride) {
    const int C = p.list[j], c = (p.alpha[C] >= 0.5 ? 3 : 0) + d;
    put(C, c, agent_load(fin + (int64_t)C * kExRec + c));
  }
  if (p.report && threadIdx.x == 0) {
    if (id == 0) p.report[0] = sweeps;
    if (!ok) p.report[1] = 1;   // (any block's; reset by ex_init_kernel)
  }
}

}  // namespace vofpc

using namespace vofpc;

extern "C" vofpc_status vofpc_extrap_opts_default(vofpc_extrap_opts *o) {
  clear_error();
  VOFPC_REQUIRE(o, VOFPC_E_INVALID_ARG, "extrap_opts_default: null argument");
  o->eps_mixed = 1e-8;
  o->layers = 2;
  o->max_iter = 120;
  o->tol = 1e-3;
  return VOFPC_OK;
}

extern "C" vofpc_status vofpc_extrapolate(vofpc_ctx ctx, vofpc_mesh M, const double *alpha, const double *T,
                                          const double *T_bface, double T_sat, const int32_t *mixed_idx,
                                          const int32_t *counts, const vofpc_interface *itf,
                                          const vofpc_extrap_opts *opts, double *gradT_l, double *gradT_v,
                                          int32_t *report) {
  clear_error();
  VOFPC_REQUIRE(ctx && M && alpha && T && T_bface && mixed_idx && counts && itf && gradT_l && gradT_v,
                VOFPC_E_INVALID_ARG, "extrapolate: null argument");
  VOFPC_REQUIRE(M->ctx && M->ctx->device == ctx->device, VOFPC_E_STATE, "extrapolate: mesh on another device");
  VOFPC_REQUIRE(itf->n && itf->A && itf->cap > 0, VOFPC_E_INVALID_ARG, "extrapolate: interface record incomplete");
  vofpc_extrap_opts o;
  if (opts) o = *opts; else vofpc_extrap_opts_default(&o);
  VOFPC_REQUIRE(o.layers >= 0 && o.layers <= 100 && o.max_iter >= 0 && o.max_iter <= 100000 && o.tol >= 0 &&
                    o.eps_mixed >= 0 && o.eps_mixed < 0.5,
                VOFPC_E_INVALID_ARG, "extrapolate: options out of range");
  VOFPC_REQUIRE(M->ncf <= INT32_MAX, VOFPC_E_INVALID_ARG, "extrapolate: more than 2^31 - 1 cell-face slots");
  VOFPC_HIP(hipSetDevice(ctx->device));
  const int64_t N = M->d.n_cells, NF = M->d.n_faces;
  hipStream_t s = ctx->stream;
  if (!M->ex_buf) {
    hipStreamCaptureStatus cs = hipStreamCaptureStatusNone;
    VOFPC_HIP(hipStreamIsCapturing(s, &cs));
    VOFPC_REQUIRE(cs == hipStreamCaptureStatusNone, VOFPC_E_STATE,
                  "extrapolate: the first call on a mesh sets up its buffers and must not be captured");
    void *a = nullptr, *b = nullptr, *c = nullptr, *d = nullptr, *e = nullptr, *f = nullptr, *g = nullptr,
         *h = nullptr, *i = nullptr, *j = nullptr;
    vofpc_status st;
    if ((st = mesh_scratch_alloc(M, (size_t)N, &a)) || (st = mesh_scratch_alloc(M, 4 * (size_t)N, &b)) ||
        (st = mesh_scratch_alloc(M, 32, &c)) || (st = mesh_scratch_alloc(M, kSyncWords * sizeof(uint32_t), &d)) ||
        (st = mesh_scratch_alloc(M, 4 * (size_t)N, &e)) || (st = mesh_scratch_alloc(M, 16 * sizeof(double) * (size_t)N, &f)) ||
        (st = mesh_scratch_alloc(M, 8 * (size_t)M->ncf, &g)) || (st = mesh_scratch_alloc(M, 8 * (size_t)N, &h)) ||
        (st = mesh_scratch_alloc(M, 4 * (size_t)M->ncf, &i)) || (st = mesh_scratch_alloc(M, 8 * (size_t)N, &j)))
      return st;
    M->ex_mark = (int8_t *)a; M->ex_list = (int32_t *)b; M->ex_info = (int32_t *)c; M->ex_flag = (uint32_t *)d;
    M->ex_entry = (int32_t *)e; M->ex_wup = (double *)g; M->ex_theta = (double *)h;
    M->ex_upn = (int32_t *)i; M->ex_upr = (int2 *)j;
    M->ex_buf = (double *)f;
  }
  const unsigned gN = (unsigned)((N + kExBlock - 1) / kExBlock);
  ex_init_kernel<<<gN, kExBlock, 0, s>>>(N, alpha, o.eps_mixed, M->ex_mark, M->ex_info, M->ex_flag, report);
  for (int l = 1; l <= o.layers; ++l)
    ring_grow_kernel<<<ring_face_blocks(NF), kRingBlock, 0, s>>>(M->d, M->ex_mark, l);
  const unsigned gL = ring_list_blocks(N);
  const unsigned gM = (unsigned)std::min<int64_t>((std::min<int64_t>(itf->cap, N) + kRingBlock - 1) / kRingBlock,
                                                  (int64_t)ctx->n_cu * 4);
  ex_list_kernel<<<gL + gM, kRingBlock, 0, s>>>(N, M->ex_mark, M->ex_list, M->ex_info + 1, (int)gL, mixed_idx, counts,
                                                *itf, M->ex_entry);
  VOFPC_HIP(hipGetLastError());
  ExParams p;
  p.m = M->d;
  p.alpha = alpha;
  p.T = T;
  p.Tb = T_bface;
  p.T_sat = T_sat;
  p.itf = *itf;
  p.list = M->ex_list;
  p.entry = M->ex_entry;
  p.info = M->ex_info;
  p.flag = M->ex_flag;
  p.mark = M->ex_mark;
  p.buf = M->ex_buf;
  p.wup = M->ex_wup;
  p.upn = M->ex_upn;
  p.upr = M->ex_upr;
  p.theta = M->ex_theta;
  p.dtau = M->min_centre_dist;
  p.tol = o.tol;
  p.max_iter = o.max_iter;
  p.gl = gradT_l;
  p.gv = gradT_v;
  p.report = report;
  // the stencil: 32 domain cells per block, four blocks per CU; the sweeps: a
  // block per CU at most, fewer for a mesh that cannot fill them
  const int64_t stencil_cells = kExBlock / kExLanes;
  const unsigned gW = (unsigned)std::max<int64_t>(
      1, std::min<int64_t>((N + stencil_cells - 1) / stencil_cells, (int64_t)ctx->n_cu * 4));
  ex_stencil_kernel<<<gW, kExBlock, 0, s>>>(p);
  const unsigned gI = (unsigned)std::max<int64_t>(
      1, std::min<int64_t>((N + kItCells - 1) / kItCells, std::min<int64_t>(ctx->n_cu, kSyncMaxBlocks)));
  ex_iterate_kernel<<<gI, kItBlock, 0, s>>>(p);
  VOFPC_HIP(hipGetLastError());
  return VOFPC_OK;
}

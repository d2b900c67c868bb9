// Cell domains grown by rings of interior face neighbours, and their lists:
// the extrapolation and the curvature chain both work on the cells within a
// few rings of the interface.
#pragma once

#include <hip/hip_runtime.h>

#include <algorithm>

#include "vofpc_internal.h"
#include "wave_ops.h"

namespace vofpc {

constexpr int kRingBlock = 256;

// faces per thread: their owners and neighbours in 16-byte loads, then every
// mark they need in flight together
constexpr int kRingRun = 4;

__device__ __forceinline__ void ring_faces(const DevMesh &m, int64_t f0, int (&o)[kRingRun], int (&q)[kRingRun]) {
  if (f0 + kRingRun <= m.n_faces) {
    const int4 ov = *reinterpret_cast<const int4 *>(m.face_owner + f0);
    const int4 qv = *reinterpret_cast<const int4 *>(m.face_neigh + f0);
    o[0] = ov.x; o[1] = ov.y; o[2] = ov.z; o[3] = ov.w;
    q[0] = qv.x; q[1] = qv.y; q[2] = qv.z; q[3] = qv.w;
  } else {
#pragma unroll
    for (int t = 0; t < kRingRun; ++t) {
      o[t] = f0 + t < m.n_faces ? m.face_owner[f0 + t] : 0;
      q[t] = f0 + t < m.n_faces ? m.face_neigh[f0 + t] : -1;
    }
  }
}

// grow the domain by one ring: neighbours of layer l-1 cells enter at layer l
// (mark: layer of each cell, -1 outside)
static __global__ __launch_bounds__(kRingBlock) void ring_grow_kernel(DevMesh m, int8_t *mark, int l) {
  const int64_t f0 = (blockIdx.x * (int64_t)kRingBlock + threadIdx.x) * kRingRun;
  if (f0 >= m.n_faces) return;
  int o[kRingRun], q[kRingRun];
  ring_faces(m, f0, o, q);
  int mo[kRingRun], mq[kRingRun];
#pragma unroll
  for (int t = 0; t < kRingRun; ++t) {
    mo[t] = mark[o[t]];
    mq[t] = q[t] >= 0 ? mark[q[t]] : 0;
  }
#pragma unroll
  for (int t = 0; t < kRingRun; ++t) {
    if (q[t] < 0) continue;
    if (mo[t] == l - 1 && mq[t] < 0) mark[q[t]] = (int8_t)l;
    if (mq[t] == l - 1 && mo[t] < 0) mark[o[t]] = (int8_t)l;
  }
}

// blocks of a launch over the faces, kRingRun a thread
static inline unsigned ring_face_blocks(int64_t n_faces) {
  const int64_t per = (int64_t)kRingBlock * kRingRun;
  return (unsigned)std::max<int64_t>(1, (n_faces + per - 1) / per);
}

// list of the cells that in_list takes (in the order of the claims: users must not
// depend on it); a tile of 16 cells a thread and one claim on the length in
// *len per block of 4,096 cells (a claim per 256 cells: 6.2 us on 195k cells,
// bound by the claims on one counter)
constexpr int kRingTile = 16;
template <class In>
static __device__ __forceinline__ void ring_list_block(int64_t n, In in_list, int32_t *list, int32_t *len,
                                                       int64_t block) {
  __shared__ int wave_tot[kRingBlock / 64];
  __shared__ int base;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int64_t c0 = block * (int64_t)kRingBlock * kRingTile;
  uint32_t in = 0;   // bit t: cell c0 + t kRingBlock + threadIdx.x
#pragma unroll
  for (int t = 0; t < kRingTile; ++t) {
    const int64_t P = c0 + t * kRingBlock + threadIdx.x;
    if (P < n && in_list(P)) in |= 1u << t;
  }
  int tot = 0;
#pragma unroll
  for (int t = 0; t < kRingTile; ++t) tot += __popcll(__ballot((in >> t) & 1));
  if (lane == 0) wave_tot[wave] = tot;
  __syncthreads();
  if (threadIdx.x == 0) {
    int all = 0;
    for (int w = 0; w < kRingBlock / 64; ++w) {
      const int c = wave_tot[w];
      wave_tot[w] = all;
      all += c;
    }
    base = all ? atomicAdd(len, all) : 0;
  }
  __syncthreads();
  int off = base + wave_tot[wave];
#pragma unroll
  for (int t = 0; t < kRingTile; ++t) {
    const uint64_t bm = __ballot((in >> t) & 1);
    if ((in >> t) & 1) list[off + lanes_below(bm)] = (int32_t)(c0 + t * kRingBlock + threadIdx.x);
    off += __popcll(bm);
  }
}

static inline unsigned ring_list_blocks(int64_t n) {
  const int64_t per = (int64_t)kRingBlock * kRingTile;
  return (unsigned)std::max<int64_t>(1, (n + per - 1) / per);
}

}  // namespace vofpc

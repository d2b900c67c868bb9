// Bracket network: per-cell features, a 32 -> 64 -> 64 -> 4 tanh perceptron
// on BF16 MFMA with FP32 accumulation (forward, backward, Adam on FP32 master
// weights), and the decoding of its output into a narrowed bisection bracket.
//
// The network predicts u = (s* - phi_min)/W (and a normal); the bracket is
// [phi_min + clamp(u,0,1) W - delta, ... + delta] with delta = k_sigma sigma W.
// The reconstruction checks the bracket and falls back, so the network only
// changes how many volume evaluations a cell needs, never its result.
//
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <new>
#include <vector>

#include "vofpc_internal.h"
#include "mlp_core.h"
#include "wave_ops.h"

namespace vofpc {

using namespace net;
constexpr float kNormalWeight = 0.1f;
constexpr int kTilesPerBlock = 4;  // 64 rows per training block

__device__ __forceinline__ void wsync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// The network of a wavefront in registers, as operands of
// v_mfma_f32_16x16x16_bf16 with the units as rows and the batch rows as
// columns: D[unit][row] = sum_k W[unit][k] in[k][row].  Lane l holds
// D[4(l/16)+j][l%16], which, rounded to BF16, is the B operand of the next
// layer for the 16 inputs those units are, so the activations never leave
// their lanes.  (Against rows as A operands staged through LDS the products
// and their order are the same: the results keep their bits.)
struct NetRegs {
  bf16x4 w1[kHid / 16][kIn / 16], w2[kHid / 16][kHid / 16], w3[kHid / 16];
  f32x4 b1[kHid / 16], b2[kHid / 16], b3;
};
constexpr int kNT = kHid / 16;   // tiles of 16 hidden units
// four consecutive floats of a caller's array (any float alignment)
typedef float f32x4u __attribute__((ext_vector_type(4), aligned(4)));

// A operand: rows r0 + l%16 (zero past nrows) of a row-major matrix with
// rows of ld values, columns k0 + 4(l/16) + j
__device__ __forceinline__ bf16x4 a_weight(const uint16_t *W, int ld, int lane, int r0, int k0, int nrows) {
  const int r = r0 + (lane & 15), k = k0 + 4 * (lane >> 4);
  bf16x4 v = {0, 0, 0, 0};
  if (r < nrows) v = *reinterpret_cast<const bf16x4 *>(W + r * ld + k);
  return v;
}

__device__ __forceinline__ void net_load(NetRegs &R, const uint16_t *wb, const float *master, int lane) {
  const int rq = 4 * (lane >> 4);
  // in the order of their use
#pragma unroll
  for (int t = 0; t < kNT; ++t) {
#pragma unroll
    for (int k = 0; k < kIn / 16; ++k) R.w1[t][k] = a_weight(wb + oW1, kIn, lane, t * 16, k * 16, kHid);
    R.b1[t] = *reinterpret_cast<const f32x4 *>(master + oB1 + t * 16 + rq);
  }
#pragma unroll
  for (int t = 0; t < kNT; ++t) {
#pragma unroll
    for (int k = 0; k < kNT; ++k) R.w2[t][k] = a_weight(wb + oW2, kHid, lane, t * 16, k * 16, kHid);
    R.b2[t] = *reinterpret_cast<const f32x4 *>(master + oB2 + t * 16 + rq);
  }
#pragma unroll
  for (int t = 0; t < kNT; ++t) R.w3[t] = a_weight(wb + oW3, kHid, lane, 0, t * 16, kOut);
  R.b3 = *reinterpret_cast<const f32x4 *>(master + oB3);
}

// four floats to BF16 (round to nearest even, the hardware's packed conversion)
__device__ __forceinline__ bf16x4 pack_bf16(f32x4 v) {
  typedef __bf16 bf16v __attribute__((ext_vector_type(4)));
  return __builtin_bit_cast(bf16x4, __builtin_convertvector(v, bf16v));
}

__device__ __forceinline__ bf16x4 activate(f32x4 z, f32x4 b) {
  f32x4 h;
#pragma unroll
  for (int j = 0; j < 4; ++j) h[j] = act_tanh(z[j] + b[j]);
  return pack_bf16(h);
}

// Inputs of batch row r0 + l%16 (zero past nr rows), columns 4(l/16) + j and
// 16 + 4(l/16) + j: two 16-byte loads a lane, whole rows a wavefront.
__device__ __forceinline__ void row_load(const float *X, int64_t r0, int nr, int lane, f32x4 (&x)[kIn / 16]) {
  const int r = lane & 15;
#pragma unroll
  for (int k = 0; k < kIn / 16; ++k) {
    x[k] = f32x4{0.f, 0.f, 0.f, 0.f};
    if (r < nr) x[k] = *reinterpret_cast<const f32x4u *>(X + (r0 + r) * kIn + k * 16 + 4 * (lane >> 4));
  }
}

// Forward pass of 16 rows; y: the four outputs of row l%16 on lanes l < 16.
__device__ __forceinline__ void tile_forward(const NetRegs &R, const f32x4 (&x)[kIn / 16], bf16x4 (&xb)[kIn / 16],
                                             bf16x4 (&h1)[kNT], bf16x4 (&h2)[kNT], f32x4 &y) {
  const f32x4 zero = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int k = 0; k < kIn / 16; ++k) xb[k] = pack_bf16(x[k]);
#pragma unroll
  for (int t = 0; t < kNT; ++t) {
    f32x4 acc = zero;
#pragma unroll
    for (int k = 0; k < kIn / 16; ++k) acc = mfma16(R.w1[t][k], xb[k], acc);
    h1[t] = activate(acc, R.b1[t]);
  }
#pragma unroll
  for (int t = 0; t < kNT; ++t) {
    f32x4 acc = zero;
#pragma unroll
    for (int k = 0; k < kNT; ++k) acc = mfma16(R.w2[t][k], h1[k], acc);
    h2[t] = activate(acc, R.b2[t]);
  }
  f32x4 acc = zero;
#pragma unroll
  for (int k = 0; k < kNT; ++k) acc = mfma16(R.w3[k], h2[k], acc);
#pragma unroll
  for (int j = 0; j < kOut; ++j) y[j] = acc[j] + R.b3[j];
}

// The rows in tiles of 16 over the wavefronts of the grid, each wavefront
// with the network in its registers and the next tile's rows in flight.
// emit(row, y) is called on the lanes that hold a row.  Bound by the vector
// ALU, the 32 tanh of a lane and tile (about 2,900 of 3,400 cycles a tile);
// the 144 bytes a row take a third of the time.  221,861 rows: 22.8 us (1.4
// TB/s), 71.9 us when each tile went through LDS with the weights re-read.
template <class Emit>
__device__ __forceinline__ void forward_rows(const float *X, int64_t n, const uint16_t *wb, const float *master,
                                             Emit emit) {
  const int lane = threadIdx.x & 63;
  const int64_t tiles = (n + 15) / 16, stride = (int64_t)gridDim.x * (blockDim.x / 64);
  int64_t t = (int64_t)blockIdx.x * (blockDim.x / 64) + (threadIdx.x >> 6);
  if (t >= tiles) return;
  NetRegs R;
  f32x4 x[kIn / 16];
  row_load(X, t * 16, (int)(n - t * 16 < 16 ? n - t * 16 : 16), lane, x);
  net_load(R, wb, master, lane);
  for (; t < tiles; t += stride) {
    const int64_t r0 = t * 16, q0 = r0 + stride * 16;
    const int nr = (int)(n - r0 < 16 ? n - r0 : 16);
    f32x4 nx[kIn / 16];
    row_load(X, q0, (int)(n - q0 < 16 ? n - q0 : 16), lane, nx);
    bf16x4 xb[kIn / 16], h1[kNT], h2[kNT];
    f32x4 y;
    tile_forward(R, x, xb, h1, h2, y);
    if (lane < nr) emit(r0 + lane, y);
#pragma unroll
    for (int k = 0; k < kIn / 16; ++k) x[k] = nx[k];
  }
}

constexpr int kNetBlock = 256;     // four wavefronts
constexpr int kNetBlocksPerCu = 3;

__global__ __launch_bounds__(kNetBlock) void mlp_forward_kernel(const float *X, int64_t n, const uint16_t *wb,
                                                                const float *master, float *Y) {
  forward_rows(X, n, wb, master, [&](int64_t r, f32x4 y) { *reinterpret_cast<f32x4u *>(Y + r * kOut) = y; });
}

// blocks of a forward launch over at most n rows
static unsigned forward_grid(vofpc_ctx ctx, int64_t n) {
  const int64_t need = ((n + 15) / 16 + kNetBlock / 64 - 1) / (kNetBlock / 64);
  return (unsigned)std::max<int64_t>(1, std::min<int64_t>(need, (int64_t)ctx->n_cu * kNetBlocksPerCu));
}

// Forward, loss and backward of the 64 rows of one block, one tile of 16 rows
// per wavefront; writes the block's partial gradient and loss (no atomics: a
// fixed-order reduction follows).  A wavefront computes its tile's
// activations and back-propagated differences in registers (the layouts of
// tile_forward serve the backward product dz1 = W2^T dz2 too) and leaves them
// in LDS with the rows innermost; then the wavefronts share out the weight
// gradients, whose products run over the rows, each sum over the block's rows
// in row order.
// Bound by the latency of one tile and of the row-ordered sums: 4,096 rows
// are 64 blocks.  A training step of 4,096 rows takes 19 us in two launches;
// one wavefront per 64 rows, scalar LDS operands, and launches of their own
// for the Adam step and the loss copy took 74 us.
constexpr int kTiles = kTilesPerBlock;
static_assert(kTiles * 64 == kNetBlock, "a wavefront per tile");
struct GradMem {
  uint16_t h1[kTiles][kHid][16], h2[kTiles][kHid][16], dz2[kTiles][kHid][16], dz1[kTiles][kHid][16];   // BF16
  uint16_t x[kTiles][kIn][16];
  float dy[kOut][kTiles * 16];
  float err[kTiles][16][kOut];
};

__device__ __forceinline__ void rows_to_lds(uint16_t (*t)[16], int u0, int row, bf16x4 v) {
#pragma unroll
  for (int j = 0; j < 4; ++j) t[u0 + j][row] = (uint16_t)v[j];
}

__global__ __launch_bounds__(kNetBlock) void mlp_grad_partial_kernel(const float *X, const float *Tg, int64_t n,
                                                                     const uint16_t *wb, const uint16_t *w2t,
                                                                     const float *master, float *partial) {
  __shared__ GradMem M;
  __shared__ float red[64];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int col = lane & 15, rq = 4 * (lane >> 4);
  const float inv_n = 1.0f / (float)n;
  {
    const int64_t r0 = ((int64_t)blockIdx.x * kTiles + wave) * 16;
    const int nr = (int)(n - r0 < 16 ? n - r0 : 16);   // may be 0 or less: a tile past the end
    f32x4 x[kIn / 16], tg = {0.f, 0.f, 0.f, 0.f};
    row_load(X, r0, nr, lane, x);
    if (lane < nr && lane < 16) tg = *reinterpret_cast<const f32x4u *>(Tg + (r0 + lane) * kOut);
    NetRegs R;
    net_load(R, wb, master, lane);
    bf16x4 wt[kNT][kNT], w3[kOut][kNT];
#pragma unroll
    for (int a = 0; a < kNT; ++a)
#pragma unroll
      for (int k = 0; k < kNT; ++k) wt[a][k] = a_weight(w2t, kHid, lane, a * 16, k * 16, kHid);
#pragma unroll
    for (int c = 0; c < kOut; ++c)
#pragma unroll
      for (int t = 0; t < kNT; ++t) w3[c][t] = *reinterpret_cast<const bf16x4 *>(wb + oW3 + c * kHid + t * 16 + rq);
    bf16x4 xb[kIn / 16], h1[kNT], h2[kNT];
    f32x4 y;
    tile_forward(R, x, xb, h1, h2, y);
    // output gradient of the mean loss, then to every lane of its row
    f32x4 d = {0.f, 0.f, 0.f, 0.f}, e = {0.f, 0.f, 0.f, 0.f};
    if (lane < 16) {
#pragma unroll
      for (int c = 0; c < kOut; ++c) {
        if (lane < nr) {
          e[c] = y[c] - tg[c];
          const float w = (c == 0) ? 1.0f : kNormalWeight;
          d[c] = 2.0f * w * e[c] * inv_n;
        }
        M.dy[c][wave * 16 + lane] = d[c];
      }
      *reinterpret_cast<f32x4 *>(&M.err[wave][lane][0]) = e;
    }
#pragma unroll
    for (int c = 0; c < kOut; ++c) d[c] = __shfl(d[c], col);
    // dz2 = (dy W3) * (1 - h2^2)   (FP32, K = 4)
    bf16x4 z2[kNT];
#pragma unroll
    for (int t = 0; t < kNT; ++t) {
      f32x4 v;
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const float h = from_bf16((uint16_t)h2[t][j]);
        float dh = 0.f;
#pragma unroll
        for (int c = 0; c < kOut; ++c) dh += d[c] * from_bf16((uint16_t)w3[c][t][j]);
        v[j] = dh * (1.0f - h * h);
      }
      z2[t] = pack_bf16(v);
    }
    // dz1 = (dz2 W2) * (1 - h1^2)
    bf16x4 z1[kNT];
#pragma unroll
    for (int t = 0; t < kNT; ++t) {
      f32x4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int k = 0; k < kNT; ++k) acc = mfma16(wt[t][k], z2[k], acc);
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const float h = from_bf16((uint16_t)h1[t][j]);
        acc[j] = acc[j] * (1.0f - h * h);
      }
      z1[t] = pack_bf16(acc);
    }
#pragma unroll
    for (int t = 0; t < kNT; ++t) {
      rows_to_lds(M.h1[wave], t * 16 + rq, col, h1[t]);
      rows_to_lds(M.h2[wave], t * 16 + rq, col, h2[t]);
      rows_to_lds(M.dz2[wave], t * 16 + rq, col, z2[t]);
      rows_to_lds(M.dz1[wave], t * 16 + rq, col, z1[t]);
    }
#pragma unroll
    for (int t = 0; t < kIn / 16; ++t) rows_to_lds(M.x[wave], t * 16 + rq, col, xb[t]);
  }
  __syncthreads();
  float *out = partial + (int64_t)blockIdx.x * (kParams + 1);
  // tiles of the block that hold rows
  const int64_t left = (n + 15) / 16 - (int64_t)blockIdx.x * kTiles;
  const int nt = left < kTiles ? (int)left : kTiles;
  auto rows4 = [&](const uint16_t (*t)[16], int u) { return *reinterpret_cast<const bf16x4 *>(&t[u][rq]); };
  // dW2 = dz2^T h1, dW1 = dz1^T x: this wavefront's 16 units, A[m][k] = dz[k][m], B[k][n] = act[k][n]
  {
    f32x4 g2[kNT], g1[kIn / 16];
#pragma unroll
    for (int b = 0; b < kNT; ++b) g2[b] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int b = 0; b < kIn / 16; ++b) g1[b] = f32x4{0.f, 0.f, 0.f, 0.f};
    for (int t = 0; t < nt; ++t) {
      const bf16x4 a2 = rows4(M.dz2[t], wave * 16 + col), a1 = rows4(M.dz1[t], wave * 16 + col);
#pragma unroll
      for (int b = 0; b < kNT; ++b) g2[b] = mfma16(a2, rows4(M.h1[t], b * 16 + col), g2[b]);
#pragma unroll
      for (int b = 0; b < kIn / 16; ++b) g1[b] = mfma16(a1, rows4(M.x[t], b * 16 + col), g1[b]);
    }
#pragma unroll
    for (int b = 0; b < kNT; ++b)
#pragma unroll
      for (int j = 0; j < 4; ++j) out[oW2 + (wave * 16 + rq + j) * kHid + b * 16 + col] = g2[b][j];
#pragma unroll
    for (int b = 0; b < kIn / 16; ++b)
#pragma unroll
      for (int j = 0; j < 4; ++j) out[oW1 + (wave * 16 + rq + j) * kIn + b * 16 + col] = g1[b][j];
  }
  // dW3 = dy^T h2, one output per wavefront, lane = hidden unit; the bias
  // sums and the loss beside it, one each
  {
    float g3 = 0.f, gb = 0.f;
    const uint16_t (*bias)[kHid][16] = wave == 0 ? M.dz2 : M.dz1;
    for (int t = 0; t < nt; ++t) {
#pragma unroll
      for (int r = 0; r < 16; ++r) g3 += M.dy[wave][t * 16 + r] * from_bf16(M.h2[t][lane][r]);
      if (wave < 2) {
#pragma unroll
        for (int r = 0; r < 16; ++r) gb += from_bf16(bias[t][lane][r]);
      } else if (wave == 2 && lane < kOut) {
#pragma unroll
        for (int r = 0; r < 16; ++r) gb += M.dy[lane][t * 16 + r];
      } else if (wave == 3) {
        const float e = M.err[t][lane / kOut][lane % kOut], w = (lane % kOut == 0) ? 1.0f : kNormalWeight;
        gb += w * e * e;
      }
    }
    out[oW3 + wave * kHid + lane] = g3;
    if (wave == 0) out[oB2 + lane] = gb;
    if (wave == 1) out[oB1 + lane] = gb;
    if (wave == 2 && lane < kOut) out[oB3 + lane] = gb;
    if (wave == 3) {
      red[lane] = gb;
      wsync();
      if (lane == 0) {
        float s = 0.f;
        for (int i = 0; i < 64; ++i) s += red[i];
        out[kParams] = s * inv_n;
      }
    }
  }
}

// Entry i of the network's parameters and its BF16 copies: row-major, and W2
// once more transposed (the backward product's operand).
__device__ __forceinline__ void store_bf16(uint16_t *wb, uint16_t *w2t, int i, float w) {
  const uint16_t h = to_bf16(w);
  wb[i] = h;
  const int k = i - oW2;
  if (k >= 0 && k < kHid * kHid) w2t[(k % kHid) * kHid + k / kHid] = h;
}

// Adam on one parameter.
struct AdamArgs {
  float *master, *m, *v;
  uint16_t *wb, *w2t;
  float lr, b1, b2, eps, bc1, bc2;
};

// Sum of the block partials in block order; the gradient and the loss go to
// the caller's arrays where given, and with `adam` each thread goes on to the
// Adam step of its parameter (a training step is this launch and the one
// before it).  The loads of a run of partials are in flight together.
__global__ __launch_bounds__(64) void mlp_reduce_kernel(const float *partial, int nblk, float *grad, float *loss,
                                                        int adam, AdamArgs p) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i > kParams) return;
  float s = 0.f;
  constexpr int kRun = 64;
  for (int b0 = 0; b0 < nblk; b0 += kRun) {
    float v[kRun];
#pragma unroll
    for (int b = 0; b < kRun; ++b) v[b] = b0 + b < nblk ? partial[(int64_t)(b0 + b) * (kParams + 1) + i] : 0.f;
#pragma unroll
    for (int b = 0; b < kRun; ++b)
      if (b0 + b < nblk) s += v[b];
  }
  if (i == kParams) {
    if (loss) *loss = s;
    return;
  }
  if (grad) grad[i] = s;
  if (!adam) return;
  const float mi = p.b1 * p.m[i] + (1.f - p.b1) * s;
  const float vi = p.b2 * p.v[i] + (1.f - p.b2) * s * s;
  p.m[i] = mi;
  p.v[i] = vi;
  const float w = p.master[i] - p.lr * (mi / p.bc1) / (sqrtf(vi / p.bc2) + p.eps);
  p.master[i] = w;
  store_bf16(p.wb, p.w2t, i, w);
}

__global__ void to_bf16_kernel(const float *src, uint16_t *wb, uint16_t *w2t) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < kParams) store_bf16(wb, w2t, i, src[i]);
}

// Decode the network output into a bracket per mixed entry.
__global__ __launch_bounds__(kNetBlock) void mlp_bracket_kernel(const float *X, const double *prange,
                                                                const int32_t *counts, int64_t cap,
                                                                const uint16_t *wb, const float *master, double ksig,
                                                                double *hlo, double *hhi) {
  int64_t n = counts[0];
  if (n > cap) n = cap;
  forward_rows(X, n, wb, master, [&](int64_t k, f32x4 y) {
    const double lo = prange[2 * k], W = prange[2 * k + 1];
    double u = (double)y[0];
    u = u < 0.0 ? 0.0 : (u > 1.0 ? 1.0 : u);
    const double sh = lo + u * W, d = ksig * W;
    const bool ok = W > 0 && !isnan(u);
    hlo[k] = ok ? sh - d : __builtin_nan("");
    hhi[k] = ok ? sh + d : __builtin_nan("");
  });
}

// ----------------------------------------------------------------- features
struct FeatMem {
  double phi[256];
  double sorted[256];
  double sum[18];
};

// 16 lanes per mixed cell, 4 cells per block.  Definitions: see the header.
// A cell is a chain of dependent gathers and reductions, and a launch of a few
// thousand cells has one wavefront per SIMD: the face data are loaded before
// the vertex field, a vertex's terms four at a time, the sums go through DPP
// and the 32 features are dealt to the lanes.  3,342 Voronoi cells: 12 us
// (15 us with one lane at the features and sums by LDS permutes); 24,431: 42 us (51).
__global__ __launch_bounds__(64) void features_kernel(DevMesh m, const double *alpha, const int32_t *mixed,
                                                      const int32_t *counts, int64_t cap, const double *phi_override,
                                                      int vertex_mode, float *feat, double *prange) {
  constexpr int W = 16, G = 4;
  __shared__ FeatMem F[G];
  const int g = threadIdx.x / W, lane = threadIdx.x % W;
  FeatMem &L = F[g];
  int64_t count = counts[0];
  if (count > cap) count = cap;
  for (int64_t k = (int64_t)blockIdx.x * G + g; k < count; k += (int64_t)gridDim.x * G) {
    const int P = mixed[k];
    const double aP = alpha[P];
    const int64_t v0 = m.cv_off[P], f0 = m.cell_face_off[P];
    const int nv = (int)(m.cv_off[P + 1] - v0), nf = (int)(m.cell_face_off[P + 1] - f0);
    const int nvv = nv < 256 ? nv : 256;
    // the lane's first face
    double S0 = 0.0, S1 = 0.0, S2 = 0.0, aQ = aP;
    bool inner = false;
    auto load_face = [&](int f) {
      const double *Sv = m.cf_S + 3 * (f0 + f);
      S0 = Sv[0]; S1 = Sv[1]; S2 = Sv[2];
      const int q = m.cf_nbr[f0 + f];
      inner = q >= 0;
      aQ = inner ? alpha[q] : aP;
    };
    if (lane < nf) load_face(lane);
    // the lane's vertices two at a time, four terms of each in flight
    for (int i = lane; i < nvv; i += 2 * W) {
      double ph[2] = {0.0, 0.0};
      int64_t j[2] = {0, 0}, j1[2] = {0, 0};
#pragma unroll
      for (int u = 0; u < 2; ++u) {
        if (i + u * W >= nvv) continue;
        const int gv = m.cv_gid[v0 + i + u * W];
        if (phi_override) {
          ph[u] = phi_override[gv];
        } else {
          j[u] = m.vc_off[gv];
          j1[u] = m.vc_off[gv + 1];
        }
      }
      const double *w = vertex_mode ? m.vc_wmean : m.vc_w;
      while (j[0] < j1[0] || j[1] < j1[1]) {
        double wt[2][4], at[2][4];
#pragma unroll
        for (int u = 0; u < 2; ++u)
#pragma unroll
          for (int t = 0; t < 4; ++t) {
            const bool in = j[u] + t < j1[u];
            wt[u][t] = in ? w[j[u] + t] : 0.0;
            at[u][t] = in ? alpha[m.vc_cell[j[u] + t]] : 0.0;
          }
#pragma unroll
        for (int u = 0; u < 2; ++u)
#pragma unroll
          for (int t = 0; t < 4; ++t, ++j[u])
            if (j[u] < j1[u]) ph[u] += wt[u][t] * at[u][t];
      }
#pragma unroll
      for (int u = 0; u < 2; ++u)
        if (i + u * W < nvv) L.phi[i + u * W] = ph[u];
    }
    wsync();
    // ranks -> sorted values
    double lmin = __builtin_inf(), lmax = -__builtin_inf(), lsum = 0;
    for (int i = lane; i < nvv; i += W) {
      const double v = L.phi[i];
      int r = 0;
#pragma unroll 4
      for (int j = 0; j < nvv; ++j) {
        const double u = L.phi[j];
        r += (u < v) || (u == v && j < i);
      }
      L.sorted[r] = v;
      lmin = fmin(lmin, v);
      lmax = fmax(lmax, v);
      lsum += v;
    }
    lmin = gmin<W>(lmin);
    lmax = gmax<W>(lmax);
    lsum = gsum<W>(lsum);
    const double pmin = lmin, Wd = lmax - lmin;
    // faces: area-weighted moments, shape tensor, neighbour alpha
    double s[18];
#pragma unroll
    for (int q = 0; q < 18; ++q) s[q] = 0.0;
    double amin = __builtin_inf(), amax = -__builtin_inf();
    for (int f = lane; f < nf; f += W) {
      if (f != lane) load_face(f);
      const double A = sqrt(S0 * S0 + S1 * S1 + S2 * S2);
      const double n0 = S0 / A, n1 = S1 / A, n2 = S2 / A;
      const double da = A * (aQ - aP);
      const double o[6] = {n0 * n0, n1 * n1, n2 * n2, n0 * n1, n0 * n2, n1 * n2};
      s[0] += A;
      s[1] += da * n0; s[2] += da * n1; s[3] += da * n2;
#pragma unroll
      for (int c = 0; c < 6; ++c) {
        s[4 + c] += da * o[c];
        s[10 + c] += A * o[c];
      }
      if (inner) {
        s[16] += aQ;
        s[17] += 1.0;
        amin = fmin(amin, aQ);
        amax = fmax(amax, aQ);
      }
    }
#pragma unroll
    for (int q = 0; q < 18; ++q) {
      s[q] = gsum<W>(s[q]);
      if (lane == 0) L.sum[q] = s[q];
    }
    amin = gmin<W>(amin);
    amax = gmax<W>(amax);
    wsync();
    auto sorted = [&](int j) { return L.sorted[j]; };
    for (int i = lane; i < 32; i += W)
      feat[k * 32 + i] = feature(i, aP, sorted, nvv, lsum, pmin, Wd, L.sum, amin, amax, nf);
    if (lane < 2) prange[2 * k + lane] = lane == 0 ? pmin : Wd;
    wsync();
  }
}

}  // namespace vofpc

using namespace vofpc;

constexpr int kW2t = (kParams + 63) / 64 * 64;   // words before the transposed W2: whole 128-byte lines

struct vofpc_mlp_s {
  vofpc_ctx ctx;
  float *master = nullptr;
  uint16_t *wb = nullptr, *w2t = nullptr;   // BF16 parameters; W2 transposed, behind them
  float *m = nullptr, *v = nullptr;
  float *partial = nullptr;
  int max_blocks = 0;
  int64_t t = 0;
};

extern "C" vofpc_status vofpc_mlp_destroy(vofpc_mlp M);

extern "C" int vofpc_mlp_param_count(void) { return kParams; }

extern "C" vofpc_status vofpc_mlp_create(vofpc_ctx ctx, int64_t max_batch, vofpc_mlp *out) {
  clear_error();
  VOFPC_REQUIRE(ctx && out && max_batch > 0, VOFPC_E_INVALID_ARG, "mlp_create: bad argument");
  *out = nullptr;
  VOFPC_HIP(hipSetDevice(ctx->device));
  vofpc_mlp M = new (std::nothrow) vofpc_mlp_s();
  VOFPC_REQUIRE(M, VOFPC_E_OOM, "mlp_create: host allocation failed");
  M->ctx = ctx;
  M->max_blocks = (int)((max_batch + 16 * kTilesPerBlock - 1) / (16 * kTilesPerBlock));
  if (hipMalloc(&M->master, sizeof(float) * kParams) != hipSuccess ||
      hipMalloc(&M->m, sizeof(float) * kParams) != hipSuccess ||
      hipMalloc(&M->v, sizeof(float) * kParams) != hipSuccess ||
      hipMalloc(&M->wb, sizeof(uint16_t) * (kW2t + kHid * kHid)) != hipSuccess ||
      hipMalloc(&M->partial, sizeof(float) * (size_t)M->max_blocks * (kParams + 1)) != hipSuccess) {
    vofpc_mlp_destroy(M);
    set_error("mlp_create: hipMalloc failed");
    return VOFPC_E_OOM;
  }
  M->w2t = M->wb + kW2t;
  VOFPC_HIP(hipMemset(M->master, 0, sizeof(float) * kParams));
  VOFPC_HIP(hipMemset(M->wb, 0, sizeof(uint16_t) * (kW2t + kHid * kHid)));
  VOFPC_HIP(hipMemset(M->m, 0, sizeof(float) * kParams));
  VOFPC_HIP(hipMemset(M->v, 0, sizeof(float) * kParams));
  M->t = 0;
  *out = M;
  return VOFPC_OK;
}

extern "C" vofpc_status vofpc_mlp_destroy(vofpc_mlp M) {
  clear_error();
  if (!M) return VOFPC_OK;
  (void)hipSetDevice(M->ctx->device);
  (void)hipFree(M->master); (void)hipFree(M->wb); (void)hipFree(M->m); (void)hipFree(M->v);
  (void)hipFree(M->partial);
  delete M;
  return VOFPC_OK;
}

extern "C" vofpc_status vofpc_mlp_set_params(vofpc_mlp M, const float *host, int64_t n) {
  clear_error();
  VOFPC_REQUIRE(M && host && n == kParams, VOFPC_E_INVALID_ARG, "mlp_set_params: need all parameters");
  VOFPC_HIP(hipSetDevice(M->ctx->device));
  VOFPC_HIP(hipMemcpy(M->master, host, sizeof(float) * kParams, hipMemcpyHostToDevice));
  VOFPC_HIP(hipMemset(M->m, 0, sizeof(float) * kParams));
  VOFPC_HIP(hipMemset(M->v, 0, sizeof(float) * kParams));
  to_bf16_kernel<<<(kParams + 255) / 256, 256, 0, M->ctx->stream>>>(M->master, M->wb, M->w2t);
  VOFPC_HIP(hipGetLastError());
  VOFPC_HIP(hipStreamSynchronize(M->ctx->stream));
  M->t = 0;
  return VOFPC_OK;
}

extern "C" vofpc_status vofpc_mlp_get_params(vofpc_mlp M, float *host, int64_t n) {
  clear_error();
  VOFPC_REQUIRE(M && host && n == kParams, VOFPC_E_INVALID_ARG, "mlp_get_params: need all parameters");
  VOFPC_HIP(hipSetDevice(M->ctx->device));
  VOFPC_HIP(hipStreamSynchronize(M->ctx->stream));
  VOFPC_HIP(hipMemcpy(host, M->master, sizeof(float) * kParams, hipMemcpyDeviceToHost));
  return VOFPC_OK;
}

extern "C" vofpc_status vofpc_mlp_forward(vofpc_ctx ctx, vofpc_mlp M, const float *X, int64_t n, float *Y) {
  clear_error();
  VOFPC_REQUIRE(ctx && M && X && Y && n > 0, VOFPC_E_INVALID_ARG, "mlp_forward: bad argument");
  VOFPC_HIP(hipSetDevice(ctx->device));
  mlp_forward_kernel<<<forward_grid(ctx, n), kNetBlock, 0, ctx->stream>>>(X, n, M->wb, M->master, Y);
  VOFPC_HIP(hipGetLastError());
  return VOFPC_OK;
}

// The gradient of the mean loss over n rows into grad and loss (either may be
// null); with `step`, Adam step number t on it.
static vofpc_status mlp_gradient(vofpc_ctx ctx, vofpc_mlp M, const float *X, const float *T, int64_t n, float *grad,
                                 float *loss, bool step, float lr) {
  const int nblk = (int)((n + 16 * kTilesPerBlock - 1) / (16 * kTilesPerBlock));
  VOFPC_REQUIRE(nblk <= M->max_blocks, VOFPC_E_INVALID_ARG, "mlp: batch larger than max_batch");
  AdamArgs p{};
  if (step) {
    M->t += 1;
    const float b1 = 0.9f, b2 = 0.999f;
    p = AdamArgs{M->master, M->m, M->v, M->wb, M->w2t, lr, b1, b2, 1e-8f, 1.0f - powf(b1, (float)M->t),
                 1.0f - powf(b2, (float)M->t)};
  }
  mlp_grad_partial_kernel<<<nblk, kNetBlock, 0, ctx->stream>>>(X, T, n, M->wb, M->w2t, M->master, M->partial);
  mlp_reduce_kernel<<<(kParams + 1 + 63) / 64, 64, 0, ctx->stream>>>(M->partial, nblk, grad, loss, step ? 1 : 0, p);
  VOFPC_HIP(hipGetLastError());
  return VOFPC_OK;
}

extern "C" vofpc_status vofpc_mlp_gradient(vofpc_ctx ctx, vofpc_mlp M, const float *X, const float *T, int64_t n,
                                           float *grad, float *loss) {
  clear_error();
  VOFPC_REQUIRE(ctx && M && X && T && n > 0, VOFPC_E_INVALID_ARG, "mlp_gradient: bad argument");
  VOFPC_HIP(hipSetDevice(ctx->device));
  return mlp_gradient(ctx, M, X, T, n, grad, loss, false, 0.f);
}

extern "C" vofpc_status vofpc_mlp_train_step(vofpc_ctx ctx, vofpc_mlp M, const float *X, const float *T, int64_t n,
                                             float lr, float *loss) {
  clear_error();
  VOFPC_REQUIRE(ctx && M && X && T && n > 0 && lr > 0, VOFPC_E_INVALID_ARG, "mlp_train_step: bad argument");
  VOFPC_HIP(hipSetDevice(ctx->device));
  return mlp_gradient(ctx, M, X, T, n, nullptr, loss, true, lr);
}

namespace vofpc {
const uint16_t *mlp_weights_bf16(vofpc_mlp M) { return M->wb; }
const float *mlp_params_f32(vofpc_mlp M) { return M->master; }
int mlp_device(vofpc_mlp M) { return M->ctx->device; }

vofpc_status launch_features(vofpc_ctx ctx, vofpc_mesh mesh, const double *alpha, const int32_t *mixed,
                             const int32_t *counts, int64_t cap, const vofpc_recon_opts *o, float *feat,
                             double *prange) {
  VOFPC_REQUIRE(alpha && mixed && counts && feat && prange && cap > 0, VOFPC_E_INVALID_ARG,
                "features: bad argument");
  VOFPC_REQUIRE(mesh->max_nv <= 256, VOFPC_E_MESH, "features: cells with more than 256 vertices");
  int64_t grid = (std::min<int64_t>(cap, mesh->d.n_cells) + 3) / 4;
  if (grid > ctx->n_cu * 16) grid = ctx->n_cu * 16;
  if (grid < 1) grid = 1;
  features_kernel<<<(unsigned)grid, 64, 0, ctx->stream>>>(mesh->d, alpha, mixed, counts, cap,
                                                          o ? o->phi_vertex : nullptr, o ? o->vertex_mode : 0, feat,
                                                          prange);
  VOFPC_HIP(hipGetLastError());
  return VOFPC_OK;
}

vofpc_status launch_bracket(vofpc_ctx ctx, vofpc_mlp M, const float *feat, const double *prange,
                            const int32_t *counts, int64_t cap, double ksig, double *hlo, double *hhi) {
  VOFPC_REQUIRE(M && feat && prange && counts && hlo && hhi && cap > 0, VOFPC_E_INVALID_ARG,
                "mlp_bracket: bad argument");
  mlp_bracket_kernel<<<forward_grid(ctx, cap), kNetBlock, 0, ctx->stream>>>(feat, prange, counts, cap, M->wb,
                                                                            M->master, ksig, hlo, hhi);
  VOFPC_HIP(hipGetLastError());
  return VOFPC_OK;
}
}  // namespace vofpc

extern "C" vofpc_status vofpc_features(vofpc_ctx ctx, vofpc_mesh mesh, const double *alpha, const int32_t *mixed_idx,
                                       const int32_t *counts, const vofpc_recon_opts *opts, float *features,
                                       double *phi_range, int64_t cap) {
  clear_error();
  VOFPC_REQUIRE(ctx && mesh, VOFPC_E_INVALID_ARG, "features: null context or mesh");
  VOFPC_HIP(hipSetDevice(ctx->device));
  return launch_features(ctx, mesh, alpha, mixed_idx, counts, cap, opts, features, phi_range);
}

extern "C" vofpc_status vofpc_mlp_bracket(vofpc_ctx ctx, vofpc_mlp M, const float *features, const double *phi_range,
                                          const int32_t *counts, int64_t cap, double delta_scale, double *hint_lo,
                                          double *hint_hi) {
  clear_error();
  VOFPC_REQUIRE(ctx, VOFPC_E_INVALID_ARG, "mlp_bracket: null context");
  VOFPC_HIP(hipSetDevice(ctx->device));
  return launch_bracket(ctx, M, features, phi_range, counts, cap, delta_scale, hint_lo, hint_hi);
}

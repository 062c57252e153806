// Learned prolongation weights: a small MLP (27 -> 64 -> 64 -> 208, ReLU, FP32) maps the
// centred log-coefficients of a coarse cell's 27 fine elements to one logit per (fine node,
// coarse corner) pair of the cell; a softmax over each node's corners gives its weights.
// Training, inference, data extraction and the assembly of per-node interpolation weights
// (averaging the predictions of all cells that share a node) run in the kernels below.
//
// A training step is one kernel for the forward pass, the L2 loss and the activation gradients and one
// for the weight gradients, both on the matrix cores in FP32 (fixed summation order, so gradients are
// deterministic); inference and the energy-norm loss run sample-parallel kernels.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <mutex>

#include "device_common.h"
#include "mlp.h"

namespace rmg {

constexpr int kMlpHalves = 14;               // half tiles of 16 output slots, the last one empty
constexpr int kMlpSlots = 16 * kMlpHalves;

// Non-corner fine nodes of a cell (x-fastest over the 4x4x4 cell nodes): position, number of
// corners, first logit, corner slots (ix + 2 iy + 4 iz).  Filled from cell_node_table.
__constant__ CellNode c_nodes[56];
__constant__ signed char c_pos2node[64];  // -1 for the 8 corners
__constant__ short c_slot_logit[kMlpSlots];       // logit of an output slot (see MlpSlots), -1 past the last
__constant__ signed char c_slot_pos[kMlpHalves][8];  // cell positions of the nodes of a half tile
__constant__ float c_kq1[64];              // Q1 Laplace element matrix of the unit cube (energy loss)

void cell_node_table(CellNode* nodes, signed char* pos2node) {
  int n = 0, off = 0;
  for (int k = 0; k < 4; ++k)
    for (int j = 0; j < 4; ++j)
      for (int i = 0; i < 4; ++i) {
        const int c[3] = {i, j, k};
        const bool corner = (i == 0 || i == 3) && (j == 0 || j == 3) && (k == 0 || k == 3);
        pos2node[(k * 4 + j) * 4 + i] = corner ? (signed char)-1 : (signed char)n;
        if (corner) continue;
        CellNode& nd = nodes[n];
        nd.pos = (k * 4 + j) * 4 + i;
        nd.first = off;
        // per axis: an interior coordinate (1, 2) interpolates from both corners, 0 / 3 from one
        int opts[3][2] = {}, no[3];
        for (int d = 0; d < 3; ++d) {
          if (c[d] == 1 || c[d] == 2) {
            opts[d][0] = 0;
            opts[d][1] = 1;
            no[d] = 2;
          } else {
            opts[d][0] = c[d] == 0 ? 0 : 1;
            no[d] = 1;
          }
        }
        int nc = 0;
        for (int iz = 0; iz < no[2]; ++iz)
          for (int iy = 0; iy < no[1]; ++iy)
            for (int ix = 0; ix < no[0]; ++ix) nd.corner[nc++] = opts[0][ix] + 2 * opts[1][iy] + 4 * opts[2][iz];
        for (int q = nc; q < 8; ++q) nd.corner[q] = 0;
        nd.ncorner = nc;
        off += nc;
        ++n;
      }
  RMG_REQUIRE(n == 56 && off == kMlpOut, RMG_ERR_ARG, "internal: cell node table");
}

// Output slots of the matrix-core kernels: the 208 logits in 13 half tiles of 16 that hold whole nodes of
// one kind, so that a lane, which holds a half tile's 16 slots of its sample, has every corner of its
// nodes: half tiles 0-3 the eight interior nodes (8 corners each), 4-9 the six faces (x low, x high, y, z;
// 4 nodes of 4 corners), 10-12 the edges along x, y, z (4 edges of 2 nodes of 2 corners, by lowest
// corner); 13 is empty.
static void mlp_slots(const CellNode* nodes, short (&logit)[kMlpSlots], signed char (&pos)[kMlpHalves][8]) {
  int filled[kMlpHalves] = {}, count[kMlpHalves] = {}, interior = 0;
  for (short& l : logit) l = -1;
  for (auto& p : pos)
    for (signed char& q : p) q = 0;
  auto put = [&](int half, const CellNode& nd, int at) {
    for (int c = 0; c < nd.ncorner; ++c) logit[half * 16 + at + c] = (short)(nd.first + c);
    pos[half][at / nd.ncorner] = (signed char)nd.pos;
    filled[half] += nd.ncorner;
    ++count[half];
  };
  for (int n = 0; n < 56; ++n) {
    const CellNode& nd = nodes[n];
    const int c[3] = {nd.pos & 3, (nd.pos >> 2) & 3, nd.pos >> 4};
    int half = 0, at = 0;
    if (nd.ncorner == 8) {
      half = interior / 2;
      at = 8 * (interior++ % 2);
    } else if (nd.ncorner == 4) {
      for (int d = 0; d < 3; ++d)
        if (c[d] == 0 || c[d] == 3) half = 4 + 2 * d + (c[d] == 3);
      at = 4 * count[half];
    } else {
      for (int d = 0; d < 3; ++d)
        if (c[d] == 1 || c[d] == 2) {
          half = 10 + d;
          const int u = c[d == 0 ? 1 : 0] == 3, v = c[d == 2 ? 1 : 2] == 3;  // the edge, lower axis first
          at = 2 * (2 * (u + 2 * v) + (c[d] == 2));
        }
    }
    put(half, nd, at);
  }
  for (int h = 0; h < kMlpHalves; ++h)
    RMG_REQUIRE(filled[h] == (h < 13 ? 16 : 0), RMG_ERR_ARG, "internal: output slots");
}

// Once per device (constant memory is per device); handles on other threads may call it too.
static void upload_tables() {
  static std::mutex mu;
  static bool done[64] = {};
  int dev = 0;
  RMG_HIP(hipGetDevice(&dev));
  RMG_REQUIRE(dev >= 0 && dev < 64, RMG_ERR_ARG, "device index beyond 63");
  std::lock_guard<std::mutex> lock(mu);
  if (done[dev]) return;
  CellNode nodes[56];
  signed char pos2node[64];
  cell_node_table(nodes, pos2node);
  RMG_HIP(hipMemcpyToSymbol(HIP_SYMBOL(c_nodes), nodes, sizeof(nodes)));
  RMG_HIP(hipMemcpyToSymbol(HIP_SYMBOL(c_pos2node), pos2node, sizeof(pos2node)));
  short logit[kMlpSlots];
  signed char pos[kMlpHalves][8];
  mlp_slots(nodes, logit, pos);
  RMG_HIP(hipMemcpyToSymbol(HIP_SYMBOL(c_slot_logit), logit, sizeof(logit)));
  RMG_HIP(hipMemcpyToSymbol(HIP_SYMBOL(c_slot_pos), pos, sizeof(pos)));
  double K[64];
  q1_laplace_element(1.0, K);
  float Kf[64];
  for (int i = 0; i < 64; ++i) Kf[i] = (float)K[i];
  RMG_HIP(hipMemcpyToSymbol(HIP_SYMBOL(c_kq1), Kf, sizeof(Kf)));
  done[dev] = true;
}

// ------------------------------------------------------------------ forward
// Parameter layout: W1 [64][27], b1 [64], W2 [64][64], b2 [64], W3 [208][64], b3 [208].
__global__ __launch_bounds__(kBlock) void k_mlp_forward(int64_t n, const float* __restrict__ X,
                                                        const float* __restrict__ th, float* __restrict__ Z,
                                                        float* __restrict__ A1, float* __restrict__ A2) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  const float* W1 = th;
  const float* b1 = W1 + kMlpH * kMlpIn;
  const float* W2 = b1 + kMlpH;
  const float* b2 = W2 + kMlpH * kMlpH;
  const float* W3 = b2 + kMlpH;
  const float* b3 = W3 + kMlpOut * kMlpH;
  // hidden activations stay in registers: every loop that indexes them is fully unrolled
  float x[kMlpIn], h1[kMlpH], h2[kMlpH];
#pragma unroll
  for (int j = 0; j < kMlpIn; ++j) x[j] = X[i * kMlpIn + j];
#pragma unroll
  for (int r = 0; r < kMlpH; ++r) {
    float a = b1[r];
#pragma unroll
    for (int j = 0; j < kMlpIn; ++j) a += W1[r * kMlpIn + j] * x[j];
    if (A1) A1[i * kMlpH + r] = a;
    h1[r] = a > 0.f ? a : 0.f;
  }
#pragma unroll
  for (int r = 0; r < kMlpH; ++r) {
    float a = b2[r];
#pragma unroll
    for (int j = 0; j < kMlpH; ++j) a += W2[r * kMlpH + j] * h1[j];
    if (A2) A2[i * kMlpH + r] = a;
    h2[r] = a > 0.f ? a : 0.f;
  }
  for (int r = 0; r < kMlpOut; ++r) {
    float a = b3[r];
#pragma unroll
    for (int j = 0; j < kMlpH; ++j) a += W3[r * kMlpH + j] * h2[j];
    Z[i * kMlpOut + r] = a;
  }
}

// Position (in the 4x4x4 cell nodes) of coarse corner slot s.
__device__ __forceinline__ int corner_pos(int s) { return 48 * ((s >> 2) & 1) + 12 * ((s >> 1) & 1) + 3 * (s & 1); }

// Softmax over the corners of node `nd` of a logit row (entries c >= nd.ncorner are left 0).
__device__ __forceinline__ void node_softmax(const float* z, const CellNode& nd, float (&w)[8]) {
  float m = z[nd.first];
#pragma unroll
  for (int c = 1; c < 8; ++c)
    if (c < nd.ncorner) m = fmaxf(m, z[nd.first + c]);
  float s = 0.f;
#pragma unroll
  for (int c = 0; c < 8; ++c) {
    w[c] = c < nd.ncorner ? expf(z[nd.first + c] - m) : 0.f;
    s += w[c];
  }
#pragma unroll
  for (int c = 0; c < 8; ++c) w[c] /= s;
}

__device__ __forceinline__ float wave_sum(float v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
  return v;
}

// Loss per sample and its gradient with respect to the logits, scaled by 1/n (the loss is a mean
// over samples), on the interpolation error delta_f = e_f - sum_c w_fc e_c (zero at the corners), in the
// energy norm: delta^T A_cell delta / (cbar sum_f e_f^2), A_cell = sum over the cell's 27 elements of
// c_e K (Q1 Laplace, unit cube), c_e = exp(X_e), cbar the mean of the c_e.  (The L2 loss,
// sum_f delta_f^2 / sum_f e_f^2, is taken where its logits are computed: k_mlp_fused.)
// One wavefront per sample: lane p holds the error at cell node p (x fastest over the 4x4x4 nodes),
// the corner values and neighbouring errors arrive by lane shuffles, and each lane of a non-corner
// node evaluates that node's softmax, so rows of E, X, Z and dZ are read and written contiguously.
// Partial sums: one per block of kMlpLossSamples.
constexpr int kMlpLossSamples = kBlock / 64;

__global__ __launch_bounds__(kBlock) void k_mlp_loss_energy(int64_t n, const float* __restrict__ Z,
                                                            const float* __restrict__ E, const float* __restrict__ X,
                                                            float* __restrict__ dZ, double* __restrict__ partials) {
  const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
  const int64_t i = (int64_t)blockIdx.x * kMlpLossSamples + wid;
  float loss = 0.f;
  if (i < n) {  // uniform over the wavefront
    const float ep = E[i * 64 + lane];
    float norm = wave_sum(ep * ep);
    if (!(norm > 0.f)) norm = 1.f;
    float ec[8];
#pragma unroll
    for (int q = 0; q < 8; ++q) ec[q] = __shfl(ep, corner_pos(q), 64);
    const int node = c_pos2node[lane];
    float w[8], ev[8], delta = 0.f;
    CellNode nd{};
    if (node >= 0) {
      nd = c_nodes[node];
      node_softmax(Z + i * kMlpOut, nd, w);
#pragma unroll
      for (int c = 0; c < 8; ++c) {
        float v = 0.f;
#pragma unroll
        for (int q = 0; q < 8; ++q) v = (c < nd.ncorner && nd.corner[c] == q) ? ec[q] : v;
        ev[c] = v;
      }
      float pred = 0.f;
#pragma unroll
      for (int c = 0; c < 8; ++c) pred += w[c] * ev[c];
      delta = ep - pred;
    }
    float g;  // d loss / d delta at this lane's node
    {
      const float ce = lane < 27 ? expf(X[i * kMlpIn + lane]) : 0.f;
      const float cbar = wave_sum(ce) * (1.0f / 27.0f);
      const int px = lane & 3, py = (lane >> 2) & 3, pz = lane >> 4;
      float ad = 0.f;  // (A_cell delta) at this node: its elements, corner roles a, neighbours b
#pragma unroll
      for (int a = 0; a < 8; ++a) {
        const int ex = px - (a & 1), ey = py - ((a >> 1) & 1), ez = pz - ((a >> 2) & 1);
        const bool valid = (unsigned)ex < 3u && (unsigned)ey < 3u && (unsigned)ez < 3u;
        const int e0x = valid ? ex : 0, e0y = valid ? ey : 0, e0z = valid ? ez : 0;
        const float c = __shfl(ce, e0x + 3 * e0y + 9 * e0z, 64);  // every lane takes part
        float sum = 0.f;
#pragma unroll
        for (int b = 0; b < 8; ++b) {
          const int nb = ((e0z + ((b >> 2) & 1)) * 4 + e0y + ((b >> 1) & 1)) * 4 + e0x + (b & 1);
          sum += c_kq1[a * 8 + b] * __shfl(delta, nb, 64);
        }
        if (valid) ad += c * sum;
      }
      const float enorm = cbar * norm;
      loss = wave_sum(delta * ad) / enorm;
      g = 2.f * ad / enorm;
    }
    if (node >= 0) {
      const float dpred = -g;
      float sdw = 0.f;
#pragma unroll
      for (int c = 0; c < 8; ++c) sdw += dpred * ev[c] * w[c];
      const float inv_n = 1.0f / (float)n;
      float* dz = dZ + i * kMlpOut;
#pragma unroll
      for (int c = 0; c < 8; ++c)
        if (c < nd.ncorner) dz[nd.first + c] = w[c] * (dpred * ev[c] - sdw) * inv_n;
    }
  }
  __shared__ float sm[kMlpLossSamples];
  if (lane == 0) sm[wid] = loss;
  __syncthreads();
  if (threadIdx.x == 0) {
    double s = 0.0;
    for (int k = 0; k < kMlpLossSamples; ++k) s += (double)sm[k];
    partials[blockIdx.x] = s;
  }
}

// Activation gradients: D2 = (dZ W3) * [A2 > 0], D1 = (D2 W2) * [A1 > 0].
__global__ __launch_bounds__(kBlock) void k_mlp_backact(int64_t n, const float* __restrict__ dZ,
                                                        const float* __restrict__ A1, const float* __restrict__ A2,
                                                        const float* __restrict__ th, float* __restrict__ D1,
                                                        float* __restrict__ D2) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  const float* W2 = th + kMlpH * kMlpIn + kMlpH;
  const float* W3 = W2 + kMlpH * kMlpH + kMlpH;
  float d2[kMlpH];
#pragma unroll
  for (int k = 0; k < kMlpH; ++k) d2[k] = 0.f;
  for (int j = 0; j < kMlpOut; ++j) {
    const float g = dZ[i * kMlpOut + j];
#pragma unroll
    for (int k = 0; k < kMlpH; ++k) d2[k] += g * W3[j * kMlpH + k];
  }
#pragma unroll
  for (int k = 0; k < kMlpH; ++k) {
    d2[k] = A2[i * kMlpH + k] > 0.f ? d2[k] : 0.f;
    D2[i * kMlpH + k] = d2[k];
  }
#pragma unroll 4
  for (int r = 0; r < kMlpH; ++r) {
    float a = 0.f;
#pragma unroll
    for (int k = 0; k < kMlpH; ++k) a += d2[k] * W2[k * kMlpH + r];
    D1[i * kMlpH + r] = A1[i * kMlpH + r] > 0.f ? a : 0.f;
  }
}

// ------------------------------------------- training step on the matrix cores
// Forward pass, loss (L2) and activation gradients of 32 samples per wavefront, FP32 throughout
// (v_mfma_f32_32x32x2_f32).  Each layer is weights times activations with a sample per column: the
// result's layout (lane = sample and half h, register i = row 8 (i / 4) + 4 h + i % 4 of a 32-row tile)
// is the next product's right operand register by register, when its reduction index runs over the rows
// in that order, so activations, logits and gradients stay in registers from the features to D1.  The
// weights lie in LDS in the order in which the products read them, 155 KB, once per block; a block of
// eight wavefronts then walks the sample tiles.  186,624 samples (the jump-coefficient training set):
// forward 589, loss 241 and activation gradients 255 us in kernels of their own on the vector units,
// 270 us here; memory's share is the 0.4 GB of activations and gradients that the weight gradients read.
using f32x16 = __attribute__((ext_vector_type(16))) float;
constexpr int kFusedThreads = 512;
constexpr int kLdsA1 = 0, kLdsA2 = kLdsA1 + 14 * 2 * 64, kLdsA3 = kLdsA2 + 32 * 2 * 64, kLdsB3 = kLdsA3 + 32 * 7 * 64,
              kLdsB2 = kLdsB3 + 112 * 2 * 64, kLdsBias = kLdsB2 + 32 * 2 * 64,
              kLdsFused = kLdsBias + kMlpH + kMlpH + kMlpSlots;
static_assert(kLdsFused * 4 <= 160 * 1024, "weights in LDS");

// Row of a 64-row layer that step s of a reduction takes in lane half h.
__device__ __forceinline__ int mfma_row(int s, int h) { return 32 * (s / 16) + 8 * (s % 16 / 4) + 4 * h + s % 4; }

__global__ __launch_bounds__(kFusedThreads) void k_mlp_fused(int64_t n, const float* __restrict__ X,
                                                             const float* __restrict__ E, const float* __restrict__ th,
                                                             float* __restrict__ A1, float* __restrict__ A2,
                                                             float* __restrict__ dZ, float* __restrict__ D1,
                                                             float* __restrict__ D2, double* __restrict__ partials) {
  __shared__ __align__(16) float w[kLdsFused];
  const float* W1 = th;
  const float* W2 = W1 + kMlpH * kMlpIn + kMlpH;
  const float* W3 = W2 + kMlpH * kMlpH + kMlpH;
  const int t = threadIdx.x, lane = t & 63, h = lane >> 5, col = lane & 31;
  for (int e = t; e < kLdsBias; e += kFusedThreads) {
    const int l = e & 63, m = l & 31, lh = l >> 5;
    float v = 0.f;
    if (e < kLdsA2) {
      const int q = e >> 6, k = 2 * (q / 2) + lh;
      if (k < kMlpIn) v = W1[(32 * (q % 2) + m) * kMlpIn + k];
    } else if (e < kLdsA3) {
      const int q = (e - kLdsA2) >> 6;
      v = W2[(32 * (q % 2) + m) * kMlpH + mfma_row(q / 2, lh)];
    } else if (e < kLdsB3) {
      const int q = (e - kLdsA3) >> 6, T = q % 7, slot = (2 * T + ((m >> 2) & 1)) * 16 + 4 * (m >> 3) + (m & 3);
      const int lg = c_slot_logit[slot];
      if (lg >= 0) v = W3[lg * kMlpH + mfma_row(q / 7, lh)];
    } else if (e < kLdsB2) {
      const int q = (e - kLdsB3) >> 6, s = q / 2, lg = c_slot_logit[(2 * (s / 16) + lh) * 16 + s % 16];
      if (lg >= 0) v = W3[lg * kMlpH + 32 * (q % 2) + m];
    } else {
      const int q = (e - kLdsB2) >> 6;
      v = W2[mfma_row(q / 2, lh) * kMlpH + 32 * (q % 2) + m];
    }
    w[e] = v;
  }
  for (int e = t; e < 2 * kMlpH + kMlpSlots; e += kFusedThreads) {
    float v;
    if (e < kMlpH) v = W1[kMlpH * kMlpIn + e];
    else if (e < 2 * kMlpH) v = W2[kMlpH * kMlpH + e - kMlpH];
    else {
      const int lg = c_slot_logit[e - 2 * kMlpH];
      v = lg >= 0 ? W3[kMlpOut * kMlpH + lg] : 0.f;
    }
    w[kLdsBias + e] = v;
  }
  __syncthreads();
  const float inv_n = 1.0f / (float)n;
  const int64_t tiles = (n + 31) / 32;
  double total = 0.0;
  // bias of a 32-row tile in the result layout, and rows of it to global memory (row-major samples)
  auto bias = [&](const float* b) __attribute__((always_inline)) {
    f32x16 c;
#pragma unroll
    for (int j = 0; j < 4; ++j)
#pragma unroll
      for (int i = 0; i < 4; ++i) c[4 * j + i] = b[8 * j + 4 * h + i];
    return c;
  };
  auto put = [&](float* row, const f32x16& c) __attribute__((always_inline)) {
#pragma unroll
    for (int j = 0; j < 4; ++j)
      *reinterpret_cast<float4*>(row + 8 * j + 4 * h) = make_float4(c[4 * j], c[4 * j + 1], c[4 * j + 2], c[4 * j + 3]);
  };
  for (int64_t tile = (int64_t)blockIdx.x * (kFusedThreads / 64) + (t >> 6); tile < tiles;
       tile += (int64_t)gridDim.x * (kFusedThreads / 64)) {
    const int64_t sample = tile * 32 + col;
    const bool live = sample < n;
    const int64_t sm = live ? sample : n - 1;
    const float* __restrict__ x = X + sm * kMlpIn;
    const float* __restrict__ e = E + sm * 64;
    float xv[14];
#pragma unroll
    for (int s = 0; s < 14; ++s) xv[s] = x[min(2 * s + h, kMlpIn - 1)];  // (past the last: weight 0)
    // half of the sample's error values each, for its norm; then its eight corners
    float norm = 0.f;
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      const float4 q = *reinterpret_cast<const float4*>(e + 32 * h + 4 * j);
      norm += q.x * q.x + q.y * q.y + (q.z * q.z + q.w * q.w);
    }
    norm += __shfl_xor(norm, 32, 64);
    if (!(norm > 0.f)) norm = 1.f;
    float ec[8];
#pragma unroll
    for (int q = 0; q < 8; ++q) ec[q] = e[corner_pos(q)];
    f32x16 a[2], b[2], g2[2];
#pragma unroll
    for (int r = 0; r < 2; ++r) a[r] = bias(w + kLdsBias + 32 * r);
#pragma unroll
    for (int s = 0; s < 14; ++s)
#pragma unroll
      for (int r = 0; r < 2; ++r)
        a[r] = __builtin_amdgcn_mfma_f32_32x32x2f32(w[kLdsA1 + (2 * s + r) * 64 + lane], xv[s], a[r], 0, 0, 0);
#pragma unroll
    for (int r = 0; r < 2; ++r) {
      if (live) put(A1 + sample * kMlpH + 32 * r, a[r]);
#pragma unroll
      for (int i = 0; i < 16; ++i) a[r][i] = fmaxf(a[r][i], 0.f);
      b[r] = bias(w + kLdsBias + kMlpH + 32 * r);
    }
#pragma unroll
    for (int s = 0; s < 32; ++s)
#pragma unroll
      for (int r = 0; r < 2; ++r)
        b[r] = __builtin_amdgcn_mfma_f32_32x32x2f32(w[kLdsA2 + (2 * s + r) * 64 + lane], a[s / 16][s % 16], b[r], 0, 0, 0);
#pragma unroll
    for (int r = 0; r < 2; ++r) {
      if (live) put(A2 + sample * kMlpH + 32 * r, b[r]);
#pragma unroll
      for (int i = 0; i < 16; ++i) {
        b[r][i] = fmaxf(b[r][i], 0.f);
        g2[r][i] = 0.f;
      }
    }
    const float scale = 2.f / norm;
    float loss = 0.f;
#pragma unroll
    for (int T = 0; T < 7; ++T) {
      f32x16 z;
#pragma unroll
      for (int j = 0; j < 4; ++j)  // (slots are half tile by half tile, so the bias row is 16 (2 T + h))
#pragma unroll
        for (int i = 0; i < 4; ++i) z[4 * j + i] = w[kLdsBias + 2 * kMlpH + 16 * (2 * T + h) + 4 * j + i];
#pragma unroll
      for (int s = 0; s < 32; ++s)
        z = __builtin_amdgcn_mfma_f32_32x32x2f32(w[kLdsA3 + (7 * s + T) * 64 + lane], b[s / 16][s % 16], z, 0, 0, 0);
      // the half tile's nodes: NC corners each
      constexpr int kNC[7] = {8, 8, 4, 4, 4, 2, 2};
      const int NC = kNC[T];
#pragma unroll
      for (int q = 0; q < 16; q += NC) {
        // corner values of this node: all, the low or high face's, or its edge's
        float ev[8], wt[8];
#pragma unroll
        for (int c = 0; c < NC; ++c) {
          if (NC == 8) {
            ev[c] = ec[c];
          } else if (NC == 4) {  // faces across axis T - 2; h: the high one
            const int d = T - 2, lo = d == 0 ? 2 * c : (d == 1 ? (c & 1) + 4 * (c >> 1) : c);
            ev[c] = h ? ec[lo + (1 << d)] : ec[lo];
          } else {  // edges along x (T 5, h 0), y (T 5, h 1), z (T 6); edge q / 4 by lowest corner
            const int g = q / 4, ex = 2 * g, ey = (g & 1) + 4 * (g >> 1), ez = g;
            if (T == 5) ev[c] = h ? ec[ey + 2 * c] : ec[ex + c];
            else ev[c] = ec[ez + 4 * c];
          }
        }
        float mx = z[q];
#pragma unroll
        for (int c = 1; c < NC; ++c) mx = fmaxf(mx, z[q + c]);
        float sum = 0.f;
#pragma unroll
        for (int c = 0; c < NC; ++c) {
          wt[c] = expf(z[q + c] - mx);
          sum += wt[c];
        }
        float pred = 0.f;
#pragma unroll
        for (int c = 0; c < NC; ++c) {
          wt[c] /= sum;
          pred += wt[c] * ev[c];
        }
        const bool node = T < 6 || h == 0;  // half tile 13 is empty
        const float delta = node ? e[c_slot_pos[2 * T + h][q / NC]] - pred : 0.f;
        loss += delta * delta;
        const float dpred = live ? -scale * delta : 0.f;
        float sdw = 0.f;
#pragma unroll
        for (int c = 0; c < NC; ++c) sdw += dpred * ev[c] * wt[c];
#pragma unroll
        for (int c = 0; c < NC; ++c) z[q + c] = wt[c] * (dpred * ev[c] - sdw) * inv_n;
      }
      if (live && (T < 6 || h == 0)) {
#pragma unroll
        for (int j = 0; j < 4; ++j)
          *reinterpret_cast<float4*>(dZ + sample * kMlpOut + 16 * (2 * T + h) + 4 * j) =
              make_float4(z[4 * j], z[4 * j + 1], z[4 * j + 2], z[4 * j + 3]);
      }
#pragma unroll
      for (int i = 0; i < 16; ++i)
#pragma unroll
        for (int r = 0; r < 2; ++r)
          g2[r] = __builtin_amdgcn_mfma_f32_32x32x2f32(w[kLdsB3 + (2 * (16 * T + i) + r) * 64 + lane], z[i], g2[r], 0, 0, 0);
    }
    loss += __shfl_xor(loss, 32, 64);
    if (live && h == 0) total += (double)(loss / norm);
    f32x16 g1[2];
#pragma unroll
    for (int r = 0; r < 2; ++r) {
#pragma unroll
      for (int i = 0; i < 16; ++i) {
        g2[r][i] = b[r][i] > 0.f ? g2[r][i] : 0.f;
        g1[r][i] = 0.f;
      }
      if (live) put(D2 + sample * kMlpH + 32 * r, g2[r]);
    }
#pragma unroll
    for (int s = 0; s < 32; ++s)
#pragma unroll
      for (int r = 0; r < 2; ++r)
        g1[r] = __builtin_amdgcn_mfma_f32_32x32x2f32(w[kLdsB2 + (2 * s + r) * 64 + lane], g2[s / 16][s % 16], g1[r], 0, 0, 0);
#pragma unroll
    for (int r = 0; r < 2; ++r) {
#pragma unroll
      for (int i = 0; i < 16; ++i) g1[r][i] = a[r][i] > 0.f ? g1[r][i] : 0.f;
      if (live) put(D1 + sample * kMlpH + 32 * r, g1[r]);
    }
  }
  // (the weights are no longer needed: their LDS holds the wavefronts' sums)
  for (int o = 32; o > 0; o >>= 1) total += __shfl_down(total, o, 64);
  __syncthreads();
  double* sums = reinterpret_cast<double*>(w);
  if (lane == 0) sums[t >> 6] = total;
  __syncthreads();
  if (t == 0) {
    double s = 0.0;
    for (int k = 0; k < kFusedThreads / 64; ++k) s += sums[k];
    partials[blockIdx.x] = s;
  }
}

// Weight gradients over a slice of samples: G[r][j] = sum_s D[s][r] H'[s][j] (H' = ReLU of the stored
// pre-activations, or the features) and the bias gradients sum_s D[s][r], on the matrix cores with two
// samples a step: the operands are rows of D and H as they lie in memory, a lane per row or column.
// Five wavefronts share a slice: three take 64 of the 208 logit rows each, one the last 16 rows and the
// first layer, one the second layer, four 32 x 32 tiles each.  FP32 sums over a slice, then FP64 over
// the slices in order (k_mlp_wgrad_reduce).  186,624 samples: 467 us in three kernels on the vector
// units, 200 us here (loading one group of steps while the other is multiplied, 768 slices instead
// of 512 or eight steps a group changed nothing, both at two wavefronts a SIMD cost 330).
constexpr int kWgBlocks = 512;
constexpr int kWgPer3 = kMlpOut * (kMlpH + 1), kWgPer2 = kMlpH * (kMlpH + 1), kWgPer1 = kMlpH * (kMlpIn + 1);
constexpr int kWgPer = kWgPer3 + kWgPer2 + kWgPer1;  // partial sums of a slice

__global__ __launch_bounds__(320) void k_mlp_wgrad(int64_t n, const float* __restrict__ X, const float* __restrict__ A1,
                                                   const float* __restrict__ A2, const float* __restrict__ dZ,
                                                   const float* __restrict__ D1, const float* __restrict__ D2,
                                                   int64_t per_block, float* __restrict__ part) {
  const int lane = threadIdx.x & 63, col = lane & 31, h = lane >> 5;
  const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int64_t s0 = (int64_t)blockIdx.x * per_block, s1 = min(n, s0 + per_block);
  float* out = part + (int64_t)blockIdx.x * kWgPer;
  f32x16 acc[2][2];
  float ab[2] = {0.f, 0.f};
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int k = 0; k < 2; ++k)
#pragma unroll
      for (int q = 0; q < 16; ++q) acc[i][k][q] = 0.f;
  constexpr int U = 4;  // steps loaded at a time
  auto tile = [&](float* o, int ld, int row0, int rows, int col0, int cols, const f32x16& c) __attribute__((always_inline)) {
#pragma unroll
    for (int q = 0; q < 16; ++q) {
      const int r = row0 + 8 * (q / 4) + 4 * h + q % 4, j = col0 + col;
      if (r < rows && j < cols) o[r * ld + j] = c[q];
    }
  };
  if (wv != 3) {
    const float* __restrict__ D = wv < 3 ? dZ + 64 * wv : D2;
    const float* __restrict__ H = wv < 3 ? A2 : A1;
    const int ld = wv < 3 ? kMlpOut : kMlpH;
    float d[2][U][2], v[2][U][2];
    // a lane's first element of D and H; groups of 2 U samples while they are whole
    const float* __restrict__ pd = D + (s0 + h) * ld + col;
    const float* __restrict__ ph = H + (s0 + h) * kMlpH + col;
    const int groups = (int)((s1 - s0) / (2 * U)), rest = (int)(s1 - s0) - groups * 2 * U;
    auto load = [&](int g, float(&dl)[U][2], float(&vl)[U][2]) __attribute__((always_inline)) {
      const float* __restrict__ qd = pd + (int64_t)min(g, groups - 1) * 2 * U * ld;
      const float* __restrict__ qh = ph + (int64_t)min(g, groups - 1) * 2 * U * kMlpH;
#pragma unroll
      for (int u = 0; u < U; ++u)
#pragma unroll
        for (int i = 0; i < 2; ++i) {
          dl[u][i] = qd[2 * u * ld + 32 * i];
          vl[u][i] = qh[2 * u * kMlpH + 32 * i];
        }
    };
    auto add = [&](const float(&dl)[U][2], const float(&vl)[U][2]) __attribute__((always_inline)) {
#pragma unroll
      for (int u = 0; u < U; ++u) {
        float b[2];
#pragma unroll
        for (int i = 0; i < 2; ++i) {
          b[i] = fmaxf(vl[u][i], 0.f);
          ab[i] += dl[u][i];
        }
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
          for (int k = 0; k < 2; ++k)
            acc[i][k] = __builtin_amdgcn_mfma_f32_32x32x2f32(dl[u][i], b[k], acc[i][k], 0, 0, 0);
      }
    };
    if (groups > 0) {
      load(0, d[0], v[0]);
      for (int g = 0; g < groups; g += 2) {  // one group loads while the other is multiplied
        load(g + 1, d[1], v[1]);
        add(d[0], v[0]);
        if (g + 1 >= groups) break;
        load(g + 2, d[0], v[0]);
        add(d[1], v[1]);
      }
    }
    if (rest > 0) {
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const bool in = 2 * u + h < rest;
        const int64_t k = in ? s0 + (int64_t)groups * 2 * U + 2 * u + h : s1 - 1;
#pragma unroll
        for (int i = 0; i < 2; ++i) {
          const float q = D[k * ld + 32 * i + col];
          d[0][u][i] = in ? q : 0.f;
          v[0][u][i] = H[k * kMlpH + 32 * i + col];
        }
      }
      add(d[0], v[0]);
    }
    float* o = wv < 3 ? out + 64 * wv * (kMlpH + 1) : out + kWgPer3;
#pragma unroll
    for (int i = 0; i < 2; ++i) {
#pragma unroll
      for (int k = 0; k < 2; ++k) tile(o, kMlpH + 1, 32 * i, 64, 32 * k, kMlpH, acc[i][k]);
      const float b = ab[i] + __shfl_xor(ab[i], 32, 64);
      if (h == 0) o[(32 * i + col) * (kMlpH + 1) + kMlpH] = b;
    }
    return;
  }
  // logit rows 192 .. 207 (columns of both halves of the second layer), and the first layer
  float ab3 = 0.f;
  const float* __restrict__ pz = dZ + (s0 + h) * kMlpOut + 192 + min(col, 15);
  const float* __restrict__ px = X + (s0 + h) * kMlpIn + min(col, kMlpIn - 1);
  const float* __restrict__ pd = D1 + (s0 + h) * kMlpH + col;
  const float* __restrict__ pv = A2 + (s0 + h) * kMlpH + col;
  const int count = (int)(s1 - s0);
  for (int s = 0; s < count; s += 2 * U) {
    float d[U][2], z[U], v[U][2], x[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const bool in = s + 2 * u + h < count;
      const int k = in ? s + 2 * u : count - 1 - h;  // (count - 1 - h >= -h: a valid sample)
      z[u] = pz[k * kMlpOut];
      x[u] = px[k * kMlpIn];
      if (!in || col > 15) z[u] = 0.f;
#pragma unroll
      for (int i = 0; i < 2; ++i) {
        d[u][i] = pd[k * kMlpH + 32 * i];
        v[u][i] = pv[k * kMlpH + 32 * i];
        if (!in) d[u][i] = 0.f;
      }
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
      ab3 += z[u];
#pragma unroll
      for (int i = 0; i < 2; ++i) {
        ab[i] += d[u][i];
        acc[0][i] = __builtin_amdgcn_mfma_f32_32x32x2f32(z[u], fmaxf(v[u][i], 0.f), acc[0][i], 0, 0, 0);
        acc[1][i] = __builtin_amdgcn_mfma_f32_32x32x2f32(d[u][i], x[u], acc[1][i], 0, 0, 0);
      }
    }
  }
  float* o1 = out + kWgPer3 + kWgPer2;
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    tile(out, kMlpH + 1, 192, kMlpOut, 32 * i, kMlpH, acc[0][i]);
    tile(o1, kMlpIn + 1, 32 * i, kMlpH, 0, kMlpIn, acc[1][i]);
    const float b = ab[i] + __shfl_xor(ab[i], 32, 64);
    if (h == 0) o1[(32 * i + col) * (kMlpIn + 1) + kMlpIn] = b;
  }
  const float b3 = ab3 + __shfl_xor(ab3, 32, 64);
  if (h == 0 && col < 16) out[(192 + col) * (kMlpH + 1) + kMlpH] = b3;
}

// Sum of the slices' partials into the flat gradient (W1, b1, W2, b2, W3, b3).  slots: the third
// layer's rows are output slots, else logits.  A block owns 64 sums; its sixteen wavefronts take
// every sixteenth slice and their sums are added in a fixed order (deterministic).
constexpr int kWgReduce = 1024;

__global__ __launch_bounds__(kWgReduce) void k_mlp_wgrad_reduce(int nblk, const float* __restrict__ part, int slots,
                                                             float* __restrict__ grad) {
  const int lane = threadIdx.x & 63, grp = threadIdx.x >> 6;
  const int t = blockIdx.x * 64 + lane;
  double s = 0.0;
  if (t < kWgPer)
    for (int b = grp; b < nblk; b += kWgReduce / 64) s += (double)part[(int64_t)b * kWgPer + t];
  __shared__ double sm[kWgReduce / 64][64];
  sm[grp][lane] = s;
  __syncthreads();
  if (grp != 0 || t >= kWgPer) return;
  double tot = 0.0;
  for (int g = 0; g < kWgReduce / 64; ++g) tot += sm[g][lane];
  constexpr int ofs2 = kMlpH * (kMlpIn + 1), ofs3 = ofs2 + kMlpH * (kMlpH + 1);
  const bool l3 = t < kWgPer3, l2 = !l3 && t < kWgPer3 + kWgPer2;
  const int u = l3 ? t : (l2 ? t - kWgPer3 : t - kWgPer3 - kWgPer2);
  const int C = l3 || l2 ? kMlpH : kMlpIn, R = l3 ? kMlpOut : kMlpH, ofs = l3 ? ofs3 : (l2 ? ofs2 : 0);
  int r = u / (C + 1);
  const int j = u - r * (C + 1);
  if (l3 && slots) r = c_slot_logit[r];
  grad[j < C ? ofs + r * C + j : ofs + R * C + r] = (float)tot;
}

__global__ void k_adam(int n, float* __restrict__ th, const float* __restrict__ g, float* __restrict__ m,
                       float* __restrict__ v, float lr, float c1, float c2) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  const float gi = g[i];
  const float mi = 0.9f * m[i] + 0.1f * gi;
  const float vi = 0.999f * v[i] + 0.001f * gi * gi;
  m[i] = mi;
  v[i] = vi;
  th[i] -= lr * (mi / c1) / (sqrtf(vi / c2) + 1e-8f);
}

// --------------------------------------------------------------- launchers
void mlp_forward(int64_t n, const float* X, const float* theta, float* Z, float* A1, float* A2, hipStream_t st) {
  if (n == 0) return;
  RMG_LAUNCH(k_mlp_forward, dim3(cdiv(n, kBlock)), dim3(kBlock), 0, st, n, X, theta, Z, A1, A2);
  LAUNCH_CHECK();
}

// Blocks of the fused training pass: one per CU, eight tiles of 32 samples at a time.
static int64_t fused_blocks(int64_t n) { return std::min<int64_t>(256, cdiv(cdiv(n, 32), kFusedThreads / 64)); }

int64_t mlp_loss_partials(int64_t n) { return std::max(cdiv(n, kMlpLossSamples), fused_blocks(n)); }

int64_t mlp_loss_energy(int64_t n, const float* Z, const float* E, const float* X, float* dZ, double* partials,
                        hipStream_t st) {
  upload_tables();
  const int64_t nb = cdiv(n, kMlpLossSamples);
  RMG_LAUNCH(k_mlp_loss_energy, dim3(nb), dim3(kBlock), 0, st, n, Z, E, X, dZ, partials);
  LAUNCH_CHECK();
  return nb;
}

int64_t mlp_fused_l2(int64_t n, const float* X, const float* E, const float* theta, float* A1, float* A2, float* dZ,
                     float* D1, float* D2, double* partials, hipStream_t st) {
  upload_tables();
  const int64_t nb = fused_blocks(n);
  RMG_LAUNCH(k_mlp_fused, dim3(nb), dim3(kFusedThreads), 0, st, n, X, E, theta, A1, A2, dZ, D1, D2, partials);
  LAUNCH_CHECK();
  return nb;
}

void mlp_backact(int64_t n, const float* dZ, const float* A1, const float* A2, const float* theta, float* D1,
                 float* D2, hipStream_t st) {
  RMG_LAUNCH(k_mlp_backact, dim3(cdiv(n, kBlock)), dim3(kBlock), 0, st, n, dZ, A1, A2, theta, D1, D2);
  LAUNCH_CHECK();
}

int64_t mlp_grad_partials() { return (int64_t)kWgBlocks * kWgPer; }

void mlp_weight_grads(int64_t n, const float* X, const float* A1, const float* A2, const float* dZ, bool slots,
                      const float* D1, const float* D2, float* grad, float* part, hipStream_t st) {
  // samples per block: a whole number of loaded steps, at most kWgBlocks blocks
  const int64_t per_block = cdiv(cdiv(n, std::min<int64_t>(kWgBlocks, cdiv(n, 64))), 16) * 16;
  const int nblk = (int)cdiv(n, per_block);
  RMG_LAUNCH(k_mlp_wgrad, dim3(nblk), dim3(320), 0, st, n, X, A1, A2, dZ, D1, D2, per_block, part);
  RMG_LAUNCH(k_mlp_wgrad_reduce, dim3(cdiv(kWgPer, 64)), dim3(kWgReduce), 0, st, nblk, part, slots ? 1 : 0, grad);
  LAUNCH_CHECK();
}

void mlp_adam(float* theta, const float* grad, float* m, float* v, int t, double lr, hipStream_t st) {
  const float c1 = (float)(1.0 - std::pow(0.9, t)), c2 = (float)(1.0 - std::pow(0.999, t));
  RMG_LAUNCH(k_adam, dim3(cdiv(kMlpParams, kBlock)), dim3(kBlock), 0, st, kMlpParams, theta, grad, m, v,
                     (float)lr, c1, c2);
  LAUNCH_CHECK();
}

// ------------------------------------------------------- data extraction
// Cells of the finest level, region by region, x-fastest; cell_off[k] = first cell of region k.
__device__ __forceinline__ int cell_region(const int64_t* __restrict__ cell_off, int nreg, int64_t c) {
  int lo = 0, hi = nreg - 1;
  while (lo < hi) {
    const int mid = (lo + hi + 1) >> 1;
    if (cell_off[mid] <= c) lo = mid;
    else hi = mid - 1;
  }
  return lo;
}

__global__ __launch_bounds__(kBlock) void k_cell_features(LevelView L, const int64_t* __restrict__ cell_off,
                                                          int64_t ncell, const float* __restrict__ logc,
                                                          float* __restrict__ X) {
  const int64_t c = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (c >= ncell) return;
  const int k = cell_region(cell_off, L.nreg, c);
  const RegionGeo R = L.regs[k];
  const int ncx = (R.ex - 1) / 3, ncy = (R.ey - 1) / 3;
  const int64_t lc = c - cell_off[k];
  const int cx = (int)(lc % ncx), cy = (int)((lc / ncx) % ncy), cz = (int)(lc / ((int64_t)ncx * ncy));
  const int ecx = L.cx - 1, ecy = L.cy - 1;
  float v[27];
  float mean = 0.f;
#pragma unroll
  for (int e = 0; e < 27; ++e) {
    const int ex = R.ox + 3 * cx + e % 3, ey = R.oy + 3 * cy + (e / 3) % 3, ez = R.oz + 3 * cz + e / 9;
    v[e] = logc ? logc[((int64_t)ez * ecy + ey) * ecx + ex] : 0.f;
    mean += v[e];
  }
  mean *= (1.0f / 27.0f);
#pragma unroll
  for (int e = 0; e < 27; ++e) X[c * kMlpIn + e] = v[e] - mean;
}

__global__ __launch_bounds__(kBlock) void k_cell_targets(LevelView L, const int64_t* __restrict__ cell_off,
                                                         int64_t ncell, const double* __restrict__ e,
                                                         float* __restrict__ E) {
  const int64_t c = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (c >= ncell) return;
  const int k = cell_region(cell_off, L.nreg, c);
  const RegionGeo R = L.regs[k];
  const int ncx = (R.ex - 1) / 3, ncy = (R.ey - 1) / 3;
  const int64_t lc = c - cell_off[k];
  const int cx = (int)(lc % ncx), cy = (int)((lc / ncx) % ncy), cz = (int)(lc / ((int64_t)ncx * ncy));
  for (int p = 0; p < 64; ++p) {
    const int x = 3 * cx + p % 4, y = 3 * cy + (p / 4) % 4, z = 3 * cz + p / 16;
    E[c * 64 + p] = (float)e[R.off + ((int64_t)z * R.ey + y) * R.ex + x];
  }
}

void cell_features(const Level& L, const int64_t* cell_off, int64_t ncell, const float* logc, float* X,
                   hipStream_t st) {
  RMG_LAUNCH(k_cell_features, dim3(cdiv(ncell, kBlock)), dim3(kBlock), 0, st, L.view(), cell_off, ncell, logc,
                     X);
  LAUNCH_CHECK();
}

void cell_targets(const Level& L, const int64_t* cell_off, int64_t ncell, const double* e, float* E, hipStream_t st) {
  RMG_LAUNCH(k_cell_targets, dim3(cdiv(ncell, kBlock)), dim3(kBlock), 0, st, L.view(), cell_off, ncell, e, E);
  LAUNCH_CHECK();
}

// ------------------------------------------------- learned weights per node
// One thread per fine node of the finest level: average the predictions of every cell (of any
// region) that contains the node, inject coarse corners, drop weights from Dirichlet coarse
// nodes to free fine nodes, and store them against the corners of the node's canonical cell.
// cellrow maps composite cells (x fastest) to logit rows.
__global__ __launch_bounds__(kBlock) void k_learned_weights(LevelView F, LevelView C, const float* __restrict__ Z,
                                                            const int* __restrict__ cellrow, double* __restrict__ pw) {
  const BlockDesc bd = F.blocks[blockIdx.x];
  const RegionGeo RF = F.regs[bd.region];
  const RegionGeo RC = C.regs[bd.region];
  const int li = bd.start + (int)threadIdx.x;
  if (li >= RF.n) return;
  int x, y, z;
  decompose(RF, li, x, y, z);
  const int gx = RF.ox + x, gy = RF.oy + y, gz = RF.oz + z;
  const int bx = min(x / 3, RC.ex - 2), by = min(y / 3, RC.ey - 2), bz = min(z / 3, RC.ez - 2);
  const int BX = RC.ox + bx, BY = RC.oy + by, BZ = RC.oz + bz;  // composite coarse index of the cell's corner 0
  double acc[8];
#pragma unroll
  for (int s = 0; s < 8; ++s) acc[s] = 0.0;
  const bool fdir = is_dirichlet(F, gx, gy, gz);
  // slots are selected, never used as array indices, so the accumulators stay in registers
  if (gx % 3 == 0 && gy % 3 == 0 && gz % 3 == 0) {
    const int s = (gx / 3 - BX) + 2 * (gy / 3 - BY) + 4 * (gz / 3 - BZ);
#pragma unroll
    for (int q = 0; q < 8; ++q) acc[q] = q == s ? 1.0 : 0.0;
  } else {
    const int ncx = (F.cx - 1) / 3, ncy = (F.cy - 1) / 3, ncz = (F.cz - 1) / 3;
    int cnt = 0;
    for (int dz = -1; dz <= 0; ++dz)
      for (int dy = -1; dy <= 0; ++dy)
        for (int dx = -1; dx <= 0; ++dx) {
          // candidate cell (composite cell index) containing the node
          const int cx = gx / 3 + dx, cy = gy / 3 + dy, cz = gz / 3 + dz;
          if (cx < 0 || cy < 0 || cz < 0 || cx >= ncx || cy >= ncy || cz >= ncz) continue;
          const int px = gx - 3 * cx, py = gy - 3 * cy, pz = gz - 3 * cz;
          if (px > 3 || py > 3 || pz > 3) continue;
          const int node = c_pos2node[(pz * 4 + py) * 4 + px];
          if (node < 0) continue;
          const CellNode nd = c_nodes[node];
          const float* zr = Z + (int64_t)cellrow[((int64_t)cz * ncy + cy) * ncx + cx] * kMlpOut;
          float w[8];
          node_softmax(zr, nd, w);
#pragma unroll
          for (int k = 0; k < 8; ++k) {
            if (k >= nd.ncorner) continue;
            const int cs = nd.corner[k];
            const int s = (cx + (cs & 1) - BX) + 2 * (cy + ((cs >> 1) & 1) - BY) + 4 * (cz + ((cs >> 2) & 1) - BZ);
#pragma unroll
            for (int q = 0; q < 8; ++q) acc[q] += q == s ? (double)w[k] : 0.0;
          }
          ++cnt;
        }
#pragma unroll
    for (int s = 0; s < 8; ++s) acc[s] /= (double)max(cnt, 1);
  }
#pragma unroll
  for (int s = 0; s < 8; ++s) {
    const int X = BX + (s & 1), Y = BY + ((s >> 1) & 1), Zc = BZ + ((s >> 2) & 1);
    double v = acc[s];
    if (!fdir && is_dirichlet(C, X, Y, Zc)) v = 0.0;
    pw[(RF.off + li) * 8 + s] = v;
  }
}

void learned_weights(const Level& F, const Level& C, const float* Z, const int* cellrow, double* pw, hipStream_t st) {
  upload_tables();
  RMG_LAUNCH(k_learned_weights, dim3(F.blocks.size()), dim3(kBlock), 0, st, F.view(), C.view(), Z, cellrow,
                     pw);
  LAUNCH_CHECK();
}

// ------------------------------------------------ stored weight validation
// Violation flags (WeightFlag): non-finite weights, support beyond the node's face, edge or
// cell, a free fine node interpolating from a Dirichlet coarse node, and weights that do not sum
// to one where no admissible corner is a dropped Dirichlet node.
__global__ __launch_bounds__(kBlock) void k_check_weights(LevelView F, LevelView C, const double* __restrict__ pw,
                                                          int* flag) {
  const BlockDesc bd = F.blocks[blockIdx.x];
  const RegionGeo RF = F.regs[bd.region];
  const RegionGeo RC = C.regs[bd.region];
  const int li = bd.start + (int)threadIdx.x;
  if (li >= RF.n) return;
  int x, y, z;
  decompose(RF, li, x, y, z);
  const int bx = min(x / 3, RC.ex - 2), by = min(y / 3, RC.ey - 2), bz = min(z / 3, RC.ez - 2);
  const int t[3] = {x - 3 * bx, y - 3 * by, z - 3 * bz};
  const bool fdir = is_dirichlet(F, RF.ox + x, RF.oy + y, RF.oz + z);
  int f = 0;
  bool dropped = false;  // some admissible corner is a Dirichlet node (its weight is dropped)
  double sum = 0.0;
  for (int s = 0; s < 8; ++s) {
    const int b[3] = {s & 1, (s >> 1) & 1, (s >> 2) & 1};
    bool admissible = true;
    for (int d = 0; d < 3; ++d)
      if ((t[d] == 0 && b[d] == 1) || (t[d] == 3 && b[d] == 0)) admissible = false;
    const bool cdir = is_dirichlet(C, RC.ox + bx + b[0], RC.oy + by + b[1], RC.oz + bz + b[2]);
    if (admissible && cdir && !fdir) dropped = true;
    const double v = pw[(RF.off + li) * 8 + s];
    if (!isfinite(v)) f |= kWeightNonFinite;
    if (v == 0.0) continue;
    sum += v;
    if (!admissible) f |= kWeightSupport;
    if (cdir && !fdir) f |= kWeightDirichlet;
  }
  if (!dropped && !(fabs(sum - 1.0) <= 1e-6)) f |= kWeightSum;
  if (f) atomicOr(flag, f);
}

// Copies of a shared node must carry the same weight for every composite coarse corner.
__global__ __launch_bounds__(kBlock) void k_check_weight_copies(LevelView F, LevelView C,
                                                                const int64_t* __restrict__ gptr,
                                                                const int* __restrict__ gcopy,
                                                                const int* __restrict__ gcomp, int64_t ng,
                                                                const double* __restrict__ pw, int* flag) {
  const int64_t g = (int64_t)blockIdx.x * kBlock + threadIdx.x;
  if (g >= ng) return;
  const int64_t ci = gcomp[g];
  const int gx = (int)(ci % F.cx), gy = (int)((ci / F.cx) % F.cy), gz = (int)(ci / ((int64_t)F.cx * F.cy));
  // composite weights of the first copy, keyed by composite corner offset from (gx/3, gy/3, gz/3) - 1
  double ref[27];
  for (int i = 0; i < 27; ++i) ref[i] = 0.0;
  for (int64_t c = gptr[g]; c < gptr[g + 1]; ++c) {
    const int gi = gcopy[c];
    int k = 0;
    while (k + 1 < F.nreg && F.regs[k + 1].off <= gi) ++k;
    const RegionGeo RF = F.regs[k], RC = C.regs[k];
    const int x = gx - RF.ox, y = gy - RF.oy, z = gz - RF.oz;
    const int bx = min(x / 3, RC.ex - 2), by = min(y / 3, RC.ey - 2), bz = min(z / 3, RC.ez - 2);
    double cur[27];
    for (int i = 0; i < 27; ++i) cur[i] = 0.0;
    for (int s = 0; s < 8; ++s) {
      const int X = RC.ox + bx + (s & 1) - gx / 3 + 1, Y = RC.oy + by + ((s >> 1) & 1) - gy / 3 + 1,
                Z = RC.oz + bz + ((s >> 2) & 1) - gz / 3 + 1;
      if ((unsigned)X > 2u || (unsigned)Y > 2u || (unsigned)Z > 2u) {
        if (pw[(int64_t)gi * 8 + s] != 0.0) atomicOr(flag, (int)kWeightSupport);
        continue;
      }
      cur[(Z * 3 + Y) * 3 + X] = pw[(int64_t)gi * 8 + s];
    }
    for (int i = 0; i < 27; ++i) {
      if (c == gptr[g]) ref[i] = cur[i];
      else if (cur[i] != ref[i]) atomicOr(flag, (int)kWeightCopies);
    }
  }
}

void check_weights(const Level& F, const Level& C, const double* pw, int* flag, hipStream_t st) {
  RMG_LAUNCH(k_check_weights, dim3(F.blocks.size()), dim3(kBlock), 0, st, F.view(), C.view(), pw, flag);
  LAUNCH_CHECK();
  if (F.ngroups > 0) {
    RMG_LAUNCH(k_check_weight_copies, dim3(cdiv(F.ngroups, kBlock)), dim3(kBlock), 0, st, F.view(), C.view(),
                       F.d_gptr.as<int64_t>(), F.d_gcopy.as<int>(), F.d_gcomp.as<int>(), F.ngroups, pw, flag);
    LAUNCH_CHECK();
  }
}

// Log of per-element coefficients (composite element grid) for the MLP features.
__global__ void k_log(int64_t n, const double* __restrict__ in, float* __restrict__ out) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) out[i] = (float)log(in[i]);
}

void launch_log(int64_t n, const double* in, float* out, hipStream_t st) {
  if (n == 0) return;
  RMG_LAUNCH(k_log, dim3(cdiv(n, kBlock)), dim3(kBlock), 0, st, n, in, out);
  LAUNCH_CHECK();
}

}  // namespace rmg

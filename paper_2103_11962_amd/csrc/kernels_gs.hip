// Region-local Gauss-Seidel (Section 3.4, Algorithm 1) for gfx950.
//
// A sweep takes the composite residual r (computed beforehand with its interface sum, the sweep's
// only communication) and, in every region k independently, visits the region's dofs in
// lexicographic order (x fastest, then y, z; the dofs of a node in order), subtracting from r_i
// the couplings A^(k)_ij delta_j to dofs already visited and setting delta_i = omega r_i / d~_i.
// That is the triangular solve (D~/omega + L_k) delta_k = r_k; a backward sweep uses the upper
// triangle in reverse order.
//
// Lexicographic order is sequential, but a node only waits for its lower neighbours, and every
// lower neighbour of (x, y, z) lies on a smaller hyperplane x + WY y + WZ z (WY = 2, WZ = 4 for
// 9- and 27-point stencils, WY = 1 for the five-point one).  The nodes of one hyperplane are
// independent, so one block per region walks the hyperplanes in order with a barrier between
// them and updates each plane's nodes in parallel: the same arithmetic as the sequential sweep.
//
// Within a plane no two nodes are neighbours in x, so reading the regional arrays would give every
// lane its own cache line.  The sweep therefore works in "slot" order: plane t of a region owns
// slots pbase[t] + q, q = (z - z0(t)) * ycand + (y - ylo(t, z)) enumerating its (z, y) candidates
// (x follows from t).  At setup the level's stencils and D~^-1 are copied into slot order
// (k_gs_fill); a sweep reads them and the neighbours' corrections by slot, which for consecutive
// lanes are consecutive.  Only r and the regional output are touched once per node in regional
// order.  The corrections are read back from the slot array written by the same block before the
// barrier (all waves of a block share the CU's vector L1, and the barrier orders the accesses).
//
// After the sweep the copies of an interface node hold different corrections (each region saw only
// its own updates); k_group_reduce<AVG> replaces them by their average, so the regional vector
// stays the regional form of a composite one.
#include <algorithm>
#include <type_traits>
#include <vector>

#include "device_common.h"

namespace rmg {

constexpr int kGsThreads = 1024;

// Hyperplanes x + wy y + 4 z = t of a region box and the slots of their nodes.
struct GsPlanes {
  static constexpr int WZ = 4;
  int ex, ey, ez, wy, ycand, tmax;
  __host__ __device__ GsPlanes(int ex_, int ey_, int ez_, int wy_) : ex(ex_), ey(ey_), ez(ez_), wy(wy_) {
    const int c = (ex - 1) / wy + 1;  // y candidates of one (t, z): y in [ylo, ylo + c)
    ycand = ey < c ? ey : c;
    tmax = (ex - 1) + wy * (ey - 1) + WZ * (ez - 1);
  }
  __host__ __device__ int z0(int t) const {
    const int n = t - (ex - 1) - wy * (ey - 1);
    return n <= 0 ? 0 : (n + WZ - 1) / WZ;
  }
  __host__ __device__ int z1(int t) const {
    const int m = t / WZ;
    return m < ez - 1 ? m : ez - 1;
  }
  __host__ __device__ int count(int t) const {
    const int a = z0(t), b = z1(t);
    return b >= a ? (b - a + 1) * ycand : 0;
  }
  __host__ __device__ int ylo(int t, int z) const {
    const int n = t - WZ * z - (ex - 1);
    return n <= 0 ? 0 : (n + wy - 1) / wy;
  }
  // node of candidate q of plane t; false if the candidate lies outside the box
  __host__ __device__ bool node(int t, int q, int& x, int& y, int& z) const {
    z = z0(t) + q / ycand;
    y = ylo(t, z) + q % ycand;
    x = t - WZ * z - wy * y;
    return y < ey && x >= 0 && x < ex;
  }
  __host__ __device__ int slot(int t, int y, int z) const { return (z - z0(t)) * ycand + (y - ylo(t, z)); }
};

template <int NPTS>
constexpr int gs_wy() {
  return NPTS == 5 ? 1 : 2;
}

// Setup: the level's stencil blocks and D~^-1 in slot order (one block per region).
template <int NPTS, int NDOF>
__global__ __launch_bounds__(kGsThreads) void k_gs_fill(LevelView L, const int* __restrict__ rplane,
                                                        const int64_t* __restrict__ pbase,
                                                        const double* __restrict__ coef,
                                                        const double* __restrict__ dinv, double* __restrict__ cs,
                                                        double* __restrict__ ds_inv) {
  constexpr int NC = NPTS * NDOF * NDOF;
  const RegionGeo R = L.regs[blockIdx.x];
  const GsPlanes P(R.ex, R.ey, R.ez, gs_wy<NPTS>());
  const int64_t* __restrict__ pb = pbase + rplane[blockIdx.x];
  for (int t = 0; t <= P.tmax; ++t) {
    const int cnt = P.count(t);
    for (int q = threadIdx.x; q < cnt; q += kGsThreads) {
      int x, y, z;
      if (!P.node(t, q, x, y, z)) continue;
      const int64_t gi = R.off + x + (int64_t)R.ex * (y + (int64_t)R.ey * z);
      const int64_t p = pb[t] + q;
      for (int c = 0; c < NC; ++c) cs[coef_index(p, c, NC)] = coef[coef_index(gi, c, NC)];
#pragma unroll
      for (int a = 0; a < NDOF; ++a) ds_inv[p * NDOF + a] = dinv[gi * NDOF + a];
    }
  }
}

template <int NPTS, int NDOF, bool BACKWARD>
__global__ __launch_bounds__(kGsThreads) void k_gs_sweep(LevelView L, const int* __restrict__ rplane,
                                                         const int64_t* __restrict__ pbase,
                                                         const double* __restrict__ cs,
                                                         const double* __restrict__ ds_inv,
                                                         const double* __restrict__ r, double* __restrict__ delta,
                                                         double* ds, double omega) {
  constexpr int NB = NDOF * NDOF;
  constexpr int NC = NPTS * NB;
  constexpr int CEN = center_index<NPTS>();
  constexpr int WY = gs_wy<NPTS>();
  const RegionGeo R = L.regs[blockIdx.x];
  const GsPlanes P(R.ex, R.ey, R.ez, WY);
  const int64_t* __restrict__ pb = pbase + rplane[blockIdx.x];
  for (int step = 0; step <= P.tmax; ++step) {
    const int t = BACKWARD ? P.tmax - step : step;
    const int cnt = P.count(t);
    for (int q = threadIdx.x; q < cnt; q += kGsThreads) {
      int x, y, z;
      if (!P.node(t, q, x, y, z)) continue;
      const int64_t gi = R.off + x + (int64_t)R.ex * (y + (int64_t)R.ey * z);
      const int64_t p = pb[t] + q;
      const double* __restrict__ c = cs + coef_index(p, 0, NC);
      double dl[NDOF];
#pragma unroll
      for (int aa = 0; aa < NDOF; ++aa) {
        const int a = BACKWARD ? NDOF - 1 - aa : aa;
        double acc = r[gi * NDOF + a];
#pragma unroll
        for (int s = BACKWARD ? CEN + 1 : 0; s < (BACKWARD ? NPTS : CEN); ++s) {
          int dx, dy, dz;
          stencil_offset<NPTS>(s, dx, dy, dz);
          if ((unsigned)(x + dx) < (unsigned)R.ex && (unsigned)(y + dy) < (unsigned)R.ey &&
              (unsigned)(z + dz) < (unsigned)R.ez) {
            const int tn = t + dx + WY * dy + GsPlanes::WZ * dz;
            const int64_t pn = pb[tn] + P.slot(tn, y + dy, z + dz);
#pragma unroll
            for (int b = 0; b < NDOF; ++b) acc -= c[(s * NB + a * NDOF + b) * kTile] * ds[pn * NDOF + b];
          }
        }
        // dofs of the same node visited before this one
#pragma unroll
        for (int b = 0; b < NDOF; ++b)
          if (BACKWARD ? b > a : b < a) acc -= c[(CEN * NB + a * NDOF + b) * kTile] * dl[b];
        dl[a] = omega * acc * ds_inv[p * NDOF + a];
      }
#pragma unroll
      for (int a = 0; a < NDOF; ++a) {
        ds[p * NDOF + a] = dl[a];
        delta[gi * NDOF + a] = dl[a];
      }
    }
    __syncthreads();
  }
}

// ------------------------------------------------------------------ 2D levels
// A sweep is one serial chain per region (ex + wy ey hyperplanes), so it is bound by the latency of
// one hyperplane, not by bytes.  Here a hyperplane costs a lane shift and a few dependent FMAs
// instead of a barrier and two dependent trips to L2: a wavefront owns 64 rows, its lane l row l,
// and at step tau computes x = tau - wy l, so the correction it needs from the row below, (x + wy - 1,
// y - 1), is lane l - 1's result of the step before (one DPP shift), and its own row's previous one
// stays in a register.  The wavefronts of a region run the same steps `lag` chunks of B steps
// apart: the last row's corrections of a wavefront reach the next one through a small LDS ring, with
// one barrier a chunk.  Couplings and D~^-1 are stored by (wavefront, step, lane) and read a whole
// chunk ahead into registers; r and the corrections pass through LDS, so that global memory sees
// runs of a row instead of one element per lane.  Same sums in the same order as k_gs_sweep, so the
// same corrections bit for bit.  234 x 241 regions (3 x 3 of them, 700 x 720 nodes), per sweep:
// five-point level 609 -> 74 us, nine-point levels 234 -> 31 us on average; multigrid to 1e-12 63.0 -> 12.0 ms.
template <int NPTS>
struct Gs2d {
  static constexpr int WY = gs_wy<NPTS>();
  static constexpr int NLOW = NPTS == 5 ? 2 : 4;  // couplings to rows and nodes visited before
  static constexpr int NV = NLOW + 1;             // with D~^-1
  // steps stored per wavefront: the last lane's last node, and one more so that the next wavefront
  // finds a (zero) correction right of the row's end
  __host__ __device__ static int steps(int ex, int ey) { return (ex + WY * ((ey < 64 ? ey : 64) - 1) + 1 + 15) / 16 * 16; }
  // stencil offset index of visited neighbour v, in summation order
  __host__ __device__ static constexpr int low(int v, bool backward) {
    return backward ? center_index<NPTS>() + 1 + v : v;
  }
};

constexpr int kGsRing = 64;  // row-end corrections in flight between two wavefronts

// Rows of a chunk's LDS slice are B + 1 apart.  Wavefronts a block may hold with chunks of B steps:
// B (NLOW + 1) couplings and B residuals are held in registers, 512 / 256 / 128 VGPRs at 4 / 8 / 16
// wavefronts, and the LDS stays below 64 KB.
constexpr int gs2d_lds(int b, int nw) { return nw * (64 * (b + 1) + kGsRing) * (int)sizeof(double); }

__device__ __forceinline__ double lane_below(double v, double lane0) {  // v of lane - 1; lane 0 takes lane0
  constexpr int kWaveShr1 = 0x138;
  const int lo = __builtin_amdgcn_update_dpp(__double2loint(lane0), __double2loint(v), kWaveShr1, 0xf, 0xf, false);
  const int hi = __builtin_amdgcn_update_dpp(__double2hiint(lane0), __double2hiint(v), kWaveShr1, 0xf, 0xf, false);
  return __hiloint2double(hi, lo);
}

__device__ __forceinline__ double lane_above(double v) {  // v of lane + 1
  constexpr int kWaveShl1 = 0x130;
  const int lo = __builtin_amdgcn_update_dpp(0, __double2loint(v), kWaveShl1, 0xf, 0xf, true);
  const int hi = __builtin_amdgcn_update_dpp(0, __double2hiint(v), kWaveShl1, 0xf, 0xf, true);
  return __hiloint2double(hi, lo);
}

// Setup: the couplings and D~^-1 of both sweep directions by (wavefront, step, lane); lanes outside
// the region hold zeros.  rec0: first record of every region; nrec records per direction.
template <int NPTS>
__global__ __launch_bounds__(kBlock) void k_gs_fill2d(LevelView L, const int64_t* __restrict__ rec0, int64_t nrec,
                                                      const double* __restrict__ coef,
                                                      const double* __restrict__ dinv, double* __restrict__ out) {
  using G = Gs2d<NPTS>;
  const RegionGeo R = L.regs[blockIdx.y];
  const int ts = G::steps(R.ex, R.ey);
  const int64_t recs = rec0[blockIdx.y + 1] - rec0[blockIdx.y];
  const int lane = threadIdx.x & 63;
  for (int64_t k = (int64_t)blockIdx.x * (kBlock / 64) + (threadIdx.x >> 6); k < recs;
       k += (int64_t)gridDim.x * (kBlock / 64)) {
    const int w = (int)(k / ts), tau = (int)(k - (int64_t)w * ts);
    const int x = tau - G::WY * lane, y = 64 * w + lane;
    const bool in = y < R.ey && (unsigned)x < (unsigned)R.ex;
    for (int back = 0; back < 2; ++back) {
      const int li = in ? (back ? R.n - 1 - (y * R.ex + x) : y * R.ex + x) : 0;
      const int64_t gi = R.off + li;
      double* o = out + ((back ? nrec : 0) + rec0[blockIdx.y] + k) * G::NV * 64 + lane;
#pragma unroll
      for (int v = 0; v < G::NLOW; ++v)
        o[v * 64] = in ? coef[coef_index(gi, back ? G::low(v, true) : G::low(v, false), NPTS)] : 0.0;
      o[G::NLOW * 64] = in ? dinv[gi] : 0.0;
    }
  }
}

template <int NPTS, bool BACKWARD, int B>
__global__ __launch_bounds__(B == 16 ? 256 : (B == 8 ? 512 : 1024)) void k_gs_sweep2d(
    LevelView L, const int64_t* __restrict__ rec0, int64_t nrec, const double* __restrict__ cs,
    const double* __restrict__ r, double* __restrict__ delta, double omega) {
  using G = Gs2d<NPTS>;
  constexpr int NV = G::NV, RPI = 64 / B;  // rows a wavefront reads or writes per instruction
  constexpr int kLag = 63 * G::WY / B + 2;  // chunks a wavefront runs behind the one below it
  extern __shared__ double lds[];
  const RegionGeo R = L.regs[blockIdx.x];
  const int lane = threadIdx.x & 63;
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int nwb = (int)blockDim.x >> 6, nw = (R.ey + 63) / 64;
  const int ts = G::steps(R.ex, R.ey), nch = ts / B;
  double* rows = lds + w * 64 * (B + 1);
  double* ring = lds + nwb * 64 * (B + 1);
  ring[w * kGsRing + lane] = 0.0;
  const double* rr = r + R.off;
  double* dd = delta + R.off;
  const double* cw =
      cs + ((BACKWARD ? nrec : 0) + rec0[blockIdx.x] + (int64_t)min(w, nw - 1) * ts) * NV * 64 + lane;
  // staged element i of this lane: row i RPI + srow, column scol of the chunk.  Lanes without a node take a
  // residual of 0 by a load out of the region's range, whatever (Inf, NaN) the residuals beside them hold:
  // D~^-1 = 0 alone would make it NaN, which the shifts carry into the rows above.
  const int srow = lane / B, scol = lane % B;
  const int y0 = 64 * w + srow, x0 = scol - G::WY * srow, l0 = y0 * R.ex + x0;
  const int di = RPI * (R.ex - G::WY);
  double cf[B][NV], rp[B], v[B];
  auto load_cf = [&](int c, int j) {
    const double* p = cw + ((int64_t)min(c, nch - 1) * B + j) * NV * 64;
#pragma unroll
    for (int k = 0; k < NV; ++k) cf[j][k] = p[k * 64];
  };
  const auto buf = __builtin_amdgcn_make_buffer_rsrc(const_cast<double*>(rr), 0, R.n * 8, 0x00020000);
  auto load_r = [&](int c) {
#pragma unroll
    for (int i = 0; i < B; ++i) {
      const int li = l0 + c * B + i * di;
      const bool in = (unsigned)(x0 + c * B - i * RPI * G::WY) < (unsigned)R.ex;
      const int at = in ? 8 * (BACKWARD ? R.n - 1 - li : li) : -256;
      rp[i] = __builtin_bit_cast(double, __builtin_amdgcn_raw_buffer_load_b64(buf, at, 0, 0));
    }
  };
#pragma unroll
  for (int j = 0; j < B; ++j) load_cf(0, j);
  load_r(0);
  __syncthreads();
  double d = 0.0, n1 = 0.0, n0 = 0.0, nm = 0.0;  // own last correction; the row below at x + 1, x, x - 1
  const int phases = nch + kLag * (nw - 1);
  for (int ph = 0; ph < phases; ++ph) {
    const int c = ph - kLag * w;
    if (w < nw && c >= 0 && c < nch) {
#pragma unroll
      for (int i = 0; i < B; ++i) rows[(i * RPI + srow) * (B + 1) + scol] = rp[i];
      load_r(c + 1);
      // lane 0 starts at x = 0 at once: the row below at x = 0 is not among its shifts
      if (G::WY == 2 && c == 0 && w > 0 && lane == 0) n1 = ring[(w - 1) * kGsRing];
      double below =
          w > 0 ? ring[(w - 1) * kGsRing + ((c * B + scol + (G::WY - 1)) & (kGsRing - 1))] : 0.0;
      __builtin_amdgcn_wave_barrier();
#pragma unroll
      for (int j = 0; j < B; ++j) v[j] = rows[lane * (B + 1) + j];
      // the chain: registers only
#pragma unroll
      for (int j = 0; j < B; ++j) {
        const double up = lane_below(d, below);
        below = lane_above(below);
        double acc = v[j];
        if constexpr (NPTS == 5) {
          if (BACKWARD) {
            acc -= cf[j][0] * d;
            acc -= cf[j][1] * up;
          } else {
            acc -= cf[j][0] * up;
            acc -= cf[j][1] * d;
          }
        } else {
          nm = n0;
          n0 = n1;
          n1 = up;
          if (BACKWARD) {
            acc -= cf[j][0] * d;
            acc -= cf[j][1] * n1;
            acc -= cf[j][2] * n0;
            acc -= cf[j][3] * nm;
          } else {
            acc -= cf[j][0] * nm;
            acc -= cf[j][1] * n0;
            acc -= cf[j][2] * n1;
            acc -= cf[j][3] * d;
          }
        }
        d = omega * acc * cf[j][G::NLOW];
        v[j] = d;
        load_cf(c + 1, j);
      }
#pragma unroll
      for (int j = 0; j < B; ++j) rows[lane * (B + 1) + j] = v[j];
      __builtin_amdgcn_wave_barrier();
#pragma unroll
      for (int i = 0; i < B; ++i) {
        const double e = rows[(i * RPI + srow) * (B + 1) + scol];
        if (y0 + i * RPI < R.ey && (unsigned)(x0 + c * B - i * RPI * G::WY) < (unsigned)R.ex) {
          const int li = l0 + c * B + i * di;
          dd[BACKWARD ? R.n - 1 - li : li] = e;
        }
      }
      if (lane < B) ring[w * kGsRing + ((c * B + lane - 63 * G::WY) & (kGsRing - 1))] = rows[63 * (B + 1) + lane];
      __builtin_amdgcn_wave_barrier();
    }
    __syncthreads();
  }
}

// The rows of every region fit sixteen wavefronts (one block; taller regions take k_gs_sweep), and
// the records, whose lanes outside the region hold zeros, stay small: below 256 MiB, or at most
// eight lanes a node (82 x 82: 3, 28 x 28: 8, 10 x 10: 20, so only a mesh of many tiny regions
// keeps k_gs_sweep for its memory).
template <int NPTS>
static bool gs2d_ok(const Level& L) {
  if (L.dim != 2 || L.ndof != 1 || L.nreg > 65535) return false;
  int64_t lanes = 0;
  for (const RegionGeo& R : L.regs) {
    if (R.ey > 1024 || (int64_t)(R.ey + 64) * R.ex >= (int64_t)1 << 28) return false;  // (byte offsets in 32 bits)
    lanes += (int64_t)((R.ey + 63) / 64) * Gs2d<NPTS>::steps(R.ex, R.ey) * 64;
  }
  return lanes <= 8 * L.n || lanes * 2 * Gs2d<NPTS>::NV * (int64_t)sizeof(double) <= (int64_t)256 << 20;
}

template <int NPTS>
static void gs2d_prepare(Level& L, hipStream_t st) {
  using G = Gs2d<NPTS>;
  std::vector<int64_t> rec0(L.nreg + 1, 0);
  int64_t most = 0;
  for (int k = 0; k < L.nreg; ++k) {
    const int64_t n = (int64_t)((L.regs[k].ey + 63) / 64) * G::steps(L.regs[k].ex, L.regs[k].ey);
    rec0[k + 1] = rec0[k] + n;
    most = std::max(most, n);
  }
  const int64_t nrec = rec0[L.nreg];
  L.gs_pbase.alloc(sizeof(int64_t) * rec0.size());
  RMG_HIP(hipMemcpyAsync(L.gs_pbase.p, rec0.data(), sizeof(int64_t) * rec0.size(), hipMemcpyHostToDevice, st));
  L.gs_coef.alloc(sizeof(double) * (size_t)(2 * nrec * G::NV * 64));
  L.gs_rplane.release();
  L.gs_dinv.release();
  L.gs_d.release();
  L.gs_records = nrec;
  const dim3 grid((unsigned)std::min<int64_t>(cdiv(most, kBlock / 64), 1024), (unsigned)L.nreg);
  RMG_LAUNCH((k_gs_fill2d<NPTS>), grid, dim3(kBlock), 0, st, L.view(), L.gs_pbase.as<int64_t>(), nrec,
             L.coef.as<double>(), L.dinv.as<double>(), L.gs_coef.as<double>());
  LAUNCH_CHECK();
  RMG_HIP(hipStreamSynchronize(st));  // the host table above is released on return
}

template <int NPTS, bool BACKWARD>
static void gs2d_launch(const Level& L, const double* r, double* delta, double omega, hipStream_t st) {
  int nw = 1;
  for (const RegionGeo& R : L.regs) nw = std::max(nw, (R.ey + 63) / 64);
  auto go = [&](auto b) {
    constexpr int B = decltype(b)::value;
    RMG_LAUNCH((k_gs_sweep2d<NPTS, BACKWARD, B>), dim3(L.nreg), dim3(64 * nw), gs2d_lds(B, nw), st, L.view(),
               L.gs_pbase.as<int64_t>(), L.gs_records, L.gs_coef.as<double>(), r, delta, omega);
  };
  if (nw <= 4) go(std::integral_constant<int, 16>());
  else if (nw <= 8) go(std::integral_constant<int, 8>());
  else go(std::integral_constant<int, 4>());
  LAUNCH_CHECK();
}
static_assert(gs2d_lds(16, 4) <= 65536 && gs2d_lds(8, 8) <= 65536 && gs2d_lds(4, 16) <= 65536, "LDS of a sweep");

template <int NPTS, int NDOF>
static void gs_fill_launch(const Level& L, hipStream_t st) {
  RMG_LAUNCH((k_gs_fill<NPTS, NDOF>), dim3(L.nreg), dim3(kGsThreads), 0, st, L.view(), L.gs_rplane.as<int>(),
                     L.gs_pbase.as<int64_t>(), L.coef.as<double>(), L.dinv.as<double>(), L.gs_coef.as<double>(),
                     L.gs_dinv.as<double>());
  LAUNCH_CHECK();
}

void launch_gs_prepare(Level& L, hipStream_t st) {
  RMG_REQUIRE(L.ndof == 1 || L.npts == 27, RMG_ERR_ARG, "internal: Gauss-Seidel blocks need 27-point levels");
  L.gs_records = 0;
  if (L.npts == 9 && gs2d_ok<9>(L)) {
    gs2d_prepare<9>(L, st);
    return;
  }
  if (L.npts == 5 && gs2d_ok<5>(L)) {
    gs2d_prepare<5>(L, st);
    return;
  }
  const int wy = L.npts == 5 ? 1 : 2;
  std::vector<int32_t> rplane(L.nreg + 1, 0);
  std::vector<int64_t> pbase;
  int64_t slots = 0;
  for (int k = 0; k < L.nreg; ++k) {
    const RegionGeo& R = L.regs[k];
    const GsPlanes P(R.ex, R.ey, R.ez, wy);
    rplane[k] = (int32_t)pbase.size();
    for (int t = 0; t <= P.tmax; ++t) {
      pbase.push_back(slots);
      slots += P.count(t);
    }
  }
  rplane[L.nreg] = (int32_t)pbase.size();
  pbase.push_back(slots);
  L.gs_rplane.alloc(sizeof(int32_t) * rplane.size());
  L.gs_pbase.alloc(sizeof(int64_t) * pbase.size());
  RMG_HIP(hipMemcpyAsync(L.gs_rplane.p, rplane.data(), sizeof(int32_t) * rplane.size(), hipMemcpyHostToDevice, st));
  RMG_HIP(hipMemcpyAsync(L.gs_pbase.p, pbase.data(), sizeof(int64_t) * pbase.size(), hipMemcpyHostToDevice, st));
  L.gs_coef.alloc(sizeof(double) * coef_elems(slots, L.ncoef()));
  L.gs_dinv.alloc(sizeof(double) * (size_t)slots * L.ndof);
  L.gs_d.alloc(sizeof(double) * (size_t)slots * L.ndof);
  if (L.npts == 27 && L.ndof == 3) gs_fill_launch<27, 3>(L, st);
  else if (L.npts == 27) gs_fill_launch<27, 1>(L, st);
  else if (L.npts == 9) gs_fill_launch<9, 1>(L, st);
  else gs_fill_launch<5, 1>(L, st);
  RMG_HIP(hipStreamSynchronize(st));  // the host tables above are released on return
}

template <int NPTS, int NDOF>
static void gs_launch(const Level& L, const double* r, double* delta, double omega, bool backward, hipStream_t st) {
  const LevelView V = L.view();
  const int* rp = L.gs_rplane.as<int>();
  const int64_t* pb = L.gs_pbase.as<int64_t>();
  const double* cs = L.gs_coef.as<double>();
  const double* di = L.gs_dinv.as<double>();
  double* ds = L.gs_d.as<double>();
  if (backward)
    RMG_LAUNCH((k_gs_sweep<NPTS, NDOF, true>), dim3(L.nreg), dim3(kGsThreads), 0, st, V, rp, pb, cs, di, r,
                       delta, ds, omega);
  else
    RMG_LAUNCH((k_gs_sweep<NPTS, NDOF, false>), dim3(L.nreg), dim3(kGsThreads), 0, st, V, rp, pb, cs, di, r,
                       delta, ds, omega);
  LAUNCH_CHECK();
}

void launch_gs_sweep(const Level& L, const double* r, double* delta, double omega, bool backward, hipStream_t st) {
  if (L.n == 0) return;
  RMG_REQUIRE(L.gs_pbase.p != nullptr, RMG_ERR_NOT_SETUP, "internal: Gauss-Seidel slot tables missing");
  if (L.gs_records > 0) {
    if (L.npts == 9) backward ? gs2d_launch<9, true>(L, r, delta, omega, st) : gs2d_launch<9, false>(L, r, delta, omega, st);
    else backward ? gs2d_launch<5, true>(L, r, delta, omega, st) : gs2d_launch<5, false>(L, r, delta, omega, st);
    return;
  }
  if (L.npts == 27 && L.ndof == 3) gs_launch<27, 3>(L, r, delta, omega, backward, st);
  else if (L.npts == 27) gs_launch<27, 1>(L, r, delta, omega, backward, st);
  else if (L.npts == 9) gs_launch<9, 1>(L, r, delta, omega, backward, st);
  else gs_launch<5, 1>(L, r, delta, omega, backward, st);
}

// Every copy of an interface dof receives the sum (AVG: the average) of the copies, summed in
// ascending region order.
template <int NDOF, bool AVG>
__global__ __launch_bounds__(kBlock) void k_group_reduce(const int64_t* __restrict__ gptr,
                                                         const int* __restrict__ gcopy, int64_t ng, double* w) {
  const int64_t g = (int64_t)blockIdx.x * kBlock + threadIdx.x;
  if (g >= ng) return;
  const int64_t a0 = gptr[g], e = gptr[g + 1];
#pragma unroll
  for (int a = 0; a < NDOF; ++a) {
    double s = 0.0;
    for (int64_t c = a0; c < e; ++c) s += w[(int64_t)gcopy[c] * NDOF + a];
    if (AVG) s *= 1.0 / (double)(e - a0);
    for (int64_t c = a0; c < e; ++c) w[(int64_t)gcopy[c] * NDOF + a] = s;
  }
}

void launch_interface_avg(const Level& L, double* w, hipStream_t st) {
  if (L.ngroups == 0) return;
  const dim3 g(cdiv(L.ngroups, kBlock));
  if (L.ndof == 3)
    RMG_LAUNCH((k_group_reduce<3, true>), g, dim3(kBlock), 0, st, L.d_gptr.as<int64_t>(),
                       L.d_gcopy.as<int>(), L.ngroups, w);
  else
    RMG_LAUNCH((k_group_reduce<1, true>), g, dim3(kBlock), 0, st, L.d_gptr.as<int64_t>(),
                       L.d_gcopy.as<int>(), L.ngroups, w);
  LAUNCH_CHECK();
}

void launch_group_reduce(const int64_t* gptr, const int* gcopy, int64_t ngroups, double* w, bool avg, hipStream_t st) {
  if (ngroups == 0) return;
  const dim3 g(cdiv(ngroups, kBlock));
  if (avg)
    RMG_LAUNCH((k_group_reduce<1, true>), g, dim3(kBlock), 0, st, gptr, gcopy, ngroups, w);
  else
    RMG_LAUNCH((k_group_reduce<1, false>), g, dim3(kBlock), 0, st, gptr, gcopy, ngroups, w);
  LAUNCH_CHECK();
}

}  // namespace rmg

// Regional stencil operations: the stencil product z = A^(k) x of every region fused with the
// node update it feeds (matvec, residual, Chebyshev step, CG product), followed by the
// interface-group kernel that sums the partial products of shared nodes over their copies in
// ascending region order (Psi^T Psi, Section 3.1 / the RegMatVec algorithm) and finishes them.
//
// Template parameters: NPTS stencil points, NDOF unknowns per node (3x3 coefficient blocks for
// elasticity), V vector type (double or float), C coefficient storage type (double, float or
// uint16_t = bfloat16; with bfloat16 the centre block comes from an FP32 array).
#include <type_traits>

#include "device_common.h"

namespace rmg {

template <class V>
struct OpP {
  const V* x;
  V* out;
  const V* b;
  const V* dinv;
  V* d;
  V c1, c2;
  const V* dinv9;  // NDOF 3 with nodal blocks: D~^-1 as one row-major 3 x 3 block per node, else null
};

// The Chebyshev / Jacobi update of the three dofs of node `node` with the nodal-block D~^-1:
// r = b - z, dd = c2 (D~^-1 r) (+ c1 dold), out = x + dd; dold the node's previous correction.
template <StencilOp OP, bool DOT, class V>
__device__ __forceinline__ double finish_block3_value(const OpP<V>& p, int64_t node, const V (&z)[3], const V (&xs)[3],
                                                      const V (&dold)[3], V (&out)[3], V (&dd)[3]) {
  const V* __restrict__ D = p.dinv9 + node * 9;
  V r[3];
#pragma unroll
  for (int a = 0; a < 3; ++a) r[a] = p.b[node * 3 + a] - z[a];
  double c = 0.0;
#pragma unroll
  for (int a = 0; a < 3; ++a) {
    const V y = D[3 * a] * r[0] + D[3 * a + 1] * r[1] + D[3 * a + 2] * r[2];
    dd[a] = p.c2 * y;
    if constexpr (OP == StencilOp::Cheb || OP == StencilOp::ChebFirst) dd[a] = fma(p.c1, dold[a], dd[a]);
    out[a] = xs[a] + dd[a];
    if constexpr (DOT) c += (double)p.b[node * 3 + a] * (double)out[a];
  }
  return c;
}

// Final update of dof i once z = (Psi^T Psi A x)_i is known; m = multiplicity of its node,
// xself = x_i: the value `out` the operation writes to p.out[i] and, for the Chebyshev steps, the
// new correction `dd`.  Returns the dof's contribution to the fused reduction, if any.
// OWN: the dof belongs to one region, whose centre coefficient `centre` is then the composite
// diagonal: the Chebyshev steps take 1 / centre (the same correctly rounded quotient as the stored
// D~^-1) instead of reading it (kOwnCentre), or are given D~^-1 itself in its place (kOwnDinv).
// The Chebyshev steps keep no direction vector: the previous correction d_(k-1) = u_(k-1) - u_(k-2)
// is the difference of the step's input and the iterate before it, which the output buffer holds
// until the step overwrites it (the cycle's two buffers alternate), so a step reads u_(k-2) in
// place of d and writes only u_k.  The step after a zero-guess start (ChebFirst) has u_(k-2) = 0
// and reads nothing for it: its previous correction is u_(k-1) itself.  `dold` is the previous
// correction (shared dofs of a Cheb step: the stencil kernel leaves it in p.d for the interface
// kernel).
constexpr int kOwnCentre = 1, kOwnDinv = 2;

template <StencilOp OP, bool DOT, class V, int OWN = 0>
__device__ __forceinline__ double finish_value(const OpP<V>& p, int64_t i, V z, int m, V xself, V centre, V dold,
                                               V& out, V& dd) {
  if constexpr (OP == StencilOp::Matvec) {
    out = z;
    return 0.0;
  } else if constexpr (OP == StencilOp::Residual) {
    out = p.b[i] - z;
    return 0.0;
  } else if constexpr (OP == StencilOp::ResidualScaled) {
    const V r = p.b[i] - z;
    out = (m == 1) ? r : r / (V)m;
    return 0.0;
  } else if constexpr (OP == StencilOp::Cheb || OP == StencilOp::ChebFirst) {
    const V bi = p.b[i];
    const V r = bi - z;
    const V di = OWN == kOwnCentre ? (V)1 / centre : (OWN == kOwnDinv ? centre : p.dinv[i]);
    dd = p.c2 * (di * r);
    dd = fma(p.c1, dold, dd);  // one rounding in every kernel
    out = xself + dd;
    if constexpr (DOT) return (double)bi * (double)out;
    return 0.0;
  } else {  // CgQ
    out = z;
    return (double)xself * (double)z;
  }
}

// The previous correction of a dof the stencil kernel finishes: x_i - u_(k-2), the latter read from
// the output buffer before it is overwritten (0 for the Jacobi steps, which have c1 = 0).
template <class V>
__device__ __forceinline__ V prev_correction(const OpP<V>& p, V xself, V uprev) {
  return p.c1 != (V)0 ? xself - uprev : (V)0;
}

// The same, written to dof i.
template <StencilOp OP, bool DOT, class V, int OWN = 0>
__device__ __forceinline__ double finish(const OpP<V>& p, int64_t i, V z, int m, V xself, V centre = (V)0) {
  V out, dd = (V)0, dold = (V)0;
  if constexpr (OP == StencilOp::Cheb) dold = prev_correction(p, xself, p.out[i]);
  if constexpr (OP == StencilOp::ChebFirst) dold = xself;
  const double c = finish_value<OP, DOT, V, OWN>(p, i, z, m, xself, centre, dold, out, dd);
  p.out[i] = out;
  return c;
}

// A shared dof's partial product goes to p.out for the interface kernel; a Chebyshev step first
// leaves its previous correction in p.d, since the partial replaces u_(k-2).
template <StencilOp OP, class V>
__device__ __forceinline__ void write_partial(const OpP<V>& p, int64_t i, V z, V xself, V uprev) {
  if constexpr (OP == StencilOp::Cheb) p.d[i] = prev_correction(p, xself, uprev);
  p.out[i] = z;
}

// The same with b_i and u_(k-2) (the output buffer's old value) already in registers (read a
// plane ahead); the arithmetic is finish_value's.
template <StencilOp OP, bool DOT, class V, int OWN = 0>
__device__ __forceinline__ double finish_pre(const OpP<V>& p, int64_t i, V z, int m, V xself, V centre, V bi, V uprev) {
  if constexpr (OP == StencilOp::Residual) {
    p.out[i] = bi - z;
    return 0.0;
  } else if constexpr (OP == StencilOp::ResidualScaled) {
    const V r = bi - z;
    p.out[i] = (m == 1) ? r : r / (V)m;
    return 0.0;
  } else if constexpr (OP == StencilOp::Cheb || OP == StencilOp::ChebFirst) {
    const V r = bi - z;
    const V di = OWN == kOwnCentre ? (V)1 / centre : (OWN == kOwnDinv ? centre : p.dinv[i]);
    V dd = p.c2 * (di * r);
    if constexpr (OP == StencilOp::Cheb) dd = fma(p.c1, prev_correction(p, xself, uprev), dd);
    if constexpr (OP == StencilOp::ChebFirst) dd = fma(p.c1, xself, dd);
    const V out = xself + dd;
    p.out[i] = out;
    if constexpr (DOT) return (double)bi * (double)out;
    return 0.0;
  } else {
    return finish<OP, DOT, V, OWN>(p, i, z, m, xself, centre);
  }
}

// Coefficient (s, a, b) of node gi; the bfloat16 storage keeps its centre block in FP32.
template <int NPTS, int NDOF, class C>
__device__ __forceinline__ auto coefv(const C* __restrict__ cf, const float* __restrict__ centre, int64_t gi, int s,
                                      int a, int b) {
  if constexpr (sizeof(C) == 2) {
    if (s == center_index<NPTS>()) return centre[gi * NDOF * NDOF + a * NDOF + b];
  }
  return CoefLoad<C>::get(cf + (s * NDOF * NDOF + a * NDOF + b) * kTile);
}

// ---------------------------------------------------------------- node-parallel
// SYM (27-point levels whose operator is symmetric): `coef` holds the upper half of each stencil,
// kSymPts blocks per node; the block of a lower offset s is the transpose of the neighbour's
// upper block at offset 26 - s, read from the neighbour's record (consecutive lanes read
// consecutive records, and the record was streamed moments before by a nearby block).
// table (27-point symmetric levels, else null): the regions' class tables, used for the
// regions whose flag in table_ok is set: a node's 27 couplings (3 x 3 blocks on 3-dof levels) are
// its class's (the values the half stencil applies, bit for bit), read from the small table
// instead of from its own and its neighbours' records.
// FUSED: the form for the small levels of k_stencil_fused.
template <int NPTS, int NDOF, class V, class C, bool SYM, bool FUSED>
__device__ __forceinline__ void node_product(const C* __restrict__ coef, const float* __restrict__ centre,
                                             const V* __restrict__ xv, const V* __restrict__ table,
                                             const int* __restrict__ table_ok, int region, const RegionGeo& R, int li,
                                             int x, int y, int z, bool inner, V (&acc)[NDOF]) {
  constexpr int NB = NDOF * NDOF;
  constexpr int NCOEF = SYM ? kSymPts * NB : NPTS * NB;
  constexpr bool kTab = NPTS == 27 && SYM;
  const int64_t gi = R.off + li;
  const V* __restrict__ xr = xv + R.off * NDOF;
  const C* __restrict__ cf = coef + coef_index(gi, 0, NCOEF);
  const int sy = R.ex, sz = R.ex * R.ey;
  const bool tabbed = kTab && table && table_ok[region];
  const V* __restrict__ tc =
      tabbed ? table + ((int64_t)region * kClasses +
                        (axis_class(z, R.ez) * 5 + axis_class(y, R.ey)) * 5 + axis_class(x, R.ex)) * kClassPts * NB
             : nullptr;
#pragma unroll
  for (int a = 0; a < NDOF; ++a) acc[a] = (V)0;
  if constexpr (NDOF == 3 && !FUSED) {
    // A block is nine loads already: one coupling block at a time, all 27 in flight would spill.  The empty
    // asm keeps the compiler from moving the two branches' last load and product behind them, where every
    // block waits for that load alone: a product on 6.1M streamed nodes 1852 us so, 1816 with a loop of
    // its own for table and stream, 1728 as it is.  (Small levels, bound by latency, are 3 to 5% faster
    // with a loop for each: below.)
#pragma unroll
    for (int s = 0; s < NPTS; ++s) {
      int dx, dy, dz;
      stencil_offset<NPTS>(s, dx, dy, dz);
      const bool ok = inner || ((unsigned)(x + dx) < (unsigned)R.ex && (unsigned)(y + dy) < (unsigned)R.ey &&
                                (unsigned)(z + dz) < (unsigned)R.ez);
      if (ok) {
        const int nb = li + dx + dy * sy + dz * sz;
        if constexpr (SYM) {
          if (kTab && tabbed) {
#pragma unroll
            for (int a = 0; a < NDOF; ++a)
#pragma unroll
              for (int b = 0; b < NDOF; ++b) acc[a] += tc[(s * NDOF + a) * NDOF + b] * xr[nb * NDOF + b];
            __asm__ volatile("");
          } else if (s >= 13) {
#pragma unroll
            for (int a = 0; a < NDOF; ++a)
#pragma unroll
              for (int b = 0; b < NDOF; ++b) {
                V c;
                if (sizeof(C) == 2 && s == 13) c = (V)centre[gi * NB + a * NDOF + b];
                else c = (V)CoefLoad<C>::get(cf + ((s - 13) * NB + a * NDOF + b) * kTile);
                acc[a] += c * xr[nb * NDOF + b];
              }
          } else {
            const C* __restrict__ cn = coef + coef_index(R.off + nb, 0, NCOEF);
#pragma unroll
            for (int a = 0; a < NDOF; ++a)
#pragma unroll
              for (int b = 0; b < NDOF; ++b)
                acc[a] += (V)CoefLoad<C>::get(cn + ((13 - s) * NB + b * NDOF + a) * kTile) * xr[nb * NDOF + b];
          }
        } else {
#pragma unroll
          for (int a = 0; a < NDOF; ++a)
#pragma unroll
            for (int b = 0; b < NDOF; ++b)
              acc[a] += (V)coefv<NPTS, NDOF, C>(cf, centre, gi, s, a, b) * xr[nb * NDOF + b];
        }
      }
    }
  } else {
    // Scalar: a coupling that leaves the box loads from the node itself and its sum is not taken, so every load is
    // unconditional and many are in flight.  (The loops over one dof keep the compiler from making branches
    // of these selections: without them a step of a small level took half as long again.)
    auto sum = [&](auto coupling) __attribute__((always_inline)) {
#pragma unroll
      for (int s = 0; s < NPTS; ++s) {
        int dx, dy, dz;
        stencil_offset<NPTS>(s, dx, dy, dz);
        const bool ok = inner || ((unsigned)(x + dx) < (unsigned)R.ex && (unsigned)(y + dy) < (unsigned)R.ey &&
                                  (unsigned)(z + dz) < (unsigned)R.ez);
        if (NDOF == 3 && !ok) continue;
        const int nb = ok ? li + dx + dy * sy + dz * sz : li;
#pragma unroll
        for (int a = 0; a < NDOF; ++a) {
          V t = acc[a];
#pragma unroll
          for (int b = 0; b < NDOF; ++b) t += coupling(s, a, b, nb) * xr[nb * NDOF + b];
          acc[a] = ok ? t : acc[a];
        }
      }
    };
    if (kTab && tabbed) {
      sum([&](int s, int a, int b, int) { return tc[(s * NDOF + a) * NDOF + b]; });
    } else if constexpr (SYM) {
      sum([&](int s, int a, int b, int nb) -> V {
        if (s > 13) return (V)CoefLoad<C>::get(cf + ((s - 13) * NB + a * NDOF + b) * kTile);
        if (s < 13)
          return (V)CoefLoad<C>::get(coef + coef_index(R.off + nb, 0, NCOEF) + ((13 - s) * NB + b * NDOF + a) * kTile);
        if (sizeof(C) == 2) return (V)centre[gi * NB + a * NDOF + b];
        return (V)CoefLoad<C>::get(cf + (a * NDOF + b) * kTile);
      });
    } else {
      sum([&](int s, int a, int b, int) { return (V)coefv<NPTS, NDOF, C>(cf, centre, gi, s, a, b); });
    }
  }
}

template <int NPTS>
__device__ __forceinline__ bool inner_node(const RegionGeo& R, int x, int y, int z) {
  return x > 0 && x < R.ex - 1 && y > 0 && y < R.ey - 1 && (NPTS != 27 || (z > 0 && z < R.ez - 1));
}

// Writes a one-region node's result; returns its contribution to the op's inner product.
template <int NDOF, StencilOp OP, bool DOT, class V>
__device__ __forceinline__ double finish_node(const OpP<V>& p, int64_t gi, const V (&acc)[NDOF], const V* xs) {
  double contrib = 0.0;
  if constexpr (NDOF == 3 && (OP == StencilOp::Cheb || OP == StencilOp::ChebFirst)) {
    if (p.dinv9) {
      V xv[3], dold[3], out[3], dd[3];
#pragma unroll
      for (int a = 0; a < 3; ++a) {
        xv[a] = xs[a];
        dold[a] = OP == StencilOp::Cheb ? prev_correction(p, xv[a], p.out[gi * 3 + a]) : xv[a];
      }
      contrib += finish_block3_value<OP, DOT, V>(p, gi, acc, xv, dold, out, dd);
#pragma unroll
      for (int a = 0; a < 3; ++a) p.out[gi * 3 + a] = out[a];
      return contrib;
    }
  }
#pragma unroll
  for (int a = 0; a < NDOF; ++a) contrib += finish<OP, DOT, V>(p, gi * NDOF + a, acc[a], 1, xs[a]);
  return contrib;
}

template <int NPTS, int NDOF, class V, class C, StencilOp OP, bool DOT, bool SYM>
__global__ __launch_bounds__(kBlock) void k_stencil(LevelView L, const C* __restrict__ coef,
                                                    const float* __restrict__ centre, OpP<V> p,
                                                    double* __restrict__ partials, const V* __restrict__ table,
                                                    const int* __restrict__ table_ok) {
  // every XCD runs a contiguous run of node blocks, so a block finds the records of the plane below
  // (its lower couplings on symmetric levels) in its own XCD's L2; its partial sum goes to the
  // node block's slot, as without the mapping
  const int blk = xcd_item((int)blockIdx.x, (int)gridDim.x);
  const BlockDesc bd = L.blocks[blk];
  const RegionGeo R = L.regs[bd.region];
  const int li = bd.start + (int)threadIdx.x;
  double contrib = 0.0;
  if (li < R.n) {
    int x, y, z;
    decompose(R, li, x, y, z);
    const int64_t gi = R.off + li;
    const V* __restrict__ xs = p.x + gi * NDOF;
    const bool inner = inner_node<NPTS>(R, x, y, z);
    V acc[NDOF];
    node_product<NPTS, NDOF, V, C, SYM, false>(coef, centre, p.x, table, table_ok, bd.region, R, li, x, y, z, inner, acc);
    if (!inner && is_shared(L, R, x, y, z)) {
#pragma unroll
      for (int a = 0; a < NDOF; ++a)  // summed over copies by k_iface
        write_partial<OP, V>(p, gi * NDOF + a, acc[a], xs[a], p.out[gi * NDOF + a]);
    } else {
      contrib = finish_node<NDOF, OP, DOT, V>(p, gi, acc, xs);
    }
  }
  if constexpr (DOT || OP == StencilOp::CgQ) {
    const double s = block_sum(contrib);
    if (threadIdx.x == 0) partials[blk] = s;
  }
}

// The same on a small level with the interface groups in the same launch: the node blocks skip the
// shared nodes, and the blocks from nb on take their copies, one per thread with a group's copies in
// one block.  A copy's product goes through LDS; every copy then sums its group's in k_iface's order,
// finishes the node from the first copy's values as k_iface does, and writes its own entry, so the
// results are k_iface's bit for bit.  Such a level is bound by the launch and by one chain of dependent
// loads (descriptor, region, couplings); the interface kernel was a second launch with a second chain.
// (Stencil and interface kernel before, this kernel now, an FP64 27-point Chebyshev step in ragged
// regions: 6,000 nodes 8.5 + 5.6 and 5.8 us, 85,000 nodes 9.4 + 5.8 and 9.2 us.)
template <int NPTS, int NDOF, class V, class C, StencilOp OP, bool DOT, bool SYM>
__global__ __launch_bounds__(kBlock) void k_stencil_fused(LevelView L, CopyView G, int nb, const C* __restrict__ coef,
                                                          const float* __restrict__ centre, OpP<V> p,
                                                          double* __restrict__ partials, const V* __restrict__ table,
                                                          const int* __restrict__ table_ok) {
  __shared__ V part[kBlock * NDOF];
  double contrib = 0.0;
  const int t = threadIdx.x;
  const int blk = (int)blockIdx.x;
  if (blk < nb) {
    const BlockDesc bd = L.blocks[blk];
    const RegionGeo R = L.regs[bd.region];
    const int li = bd.start + t;
    if (li < R.n) {
      int x, y, z;
      decompose(R, li, x, y, z);
      const bool inner = inner_node<NPTS>(R, x, y, z);
      if (inner || !is_shared(L, R, x, y, z)) {
        const int64_t gi = R.off + li;
        V acc[NDOF];
        node_product<NPTS, NDOF, V, C, SYM, true>(coef, centre, p.x, table, table_ok, bd.region, R, li, x, y, z, inner, acc);
        contrib = finish_node<NDOF, OP, DOT, V>(p, gi, acc, p.x + gi * NDOF);
      }
    }
  } else {
    const int first = G.start[blk - nb], cnt = G.start[blk - nb + 1] - first;
    int4 ci = make_int4(0, 0, 0, 0);
    int64_t n0 = 0;  // the group's first copy
    V uprev[NDOF];
#pragma unroll
    for (int a = 0; a < NDOF; ++a) uprev[a] = (V)0;
    if (t < cnt) {
      ci = G.info[first + t];
      n0 = G.info[first + ci.z].x;
      const RegionGeo R = L.regs[ci.y];
      const int li = (int)(ci.x - R.off);
      int x, y, z;
      decompose(R, li, x, y, z);
      V acc[NDOF];
      node_product<NPTS, NDOF, V, C, SYM, true>(coef, centre, p.x, table, table_ok, ci.y, R, li, x, y, z, false, acc);
#pragma unroll
      for (int a = 0; a < NDOF; ++a) {
        part[t * NDOF + a] = acc[a];
        if constexpr (OP == StencilOp::Cheb) uprev[a] = p.out[n0 * NDOF + a];  // before the first copy writes it
      }
    }
    __syncthreads();
    if (t < cnt) {
      V z[NDOF], xs[NDOF], dold[NDOF], out[NDOF], dd[NDOF];
#pragma unroll
      for (int a = 0; a < NDOF; ++a) {
        V s = (V)0;
        for (int k = ci.z; k < ci.z + ci.w; ++k) s += part[k * NDOF + a];
        z[a] = s;
        xs[a] = p.x[n0 * NDOF + a];
        dold[a] = OP == StencilOp::Cheb ? prev_correction(p, xs[a], uprev[a]) : xs[a];
        dd[a] = (V)0;
      }
      bool block = false;
      double c = 0.0;
      if constexpr (NDOF == 3 && (OP == StencilOp::Cheb || OP == StencilOp::ChebFirst)) {
        if (p.dinv9) {
          c = finish_block3_value<OP, DOT, V>(p, n0, z, xs, dold, out, dd);
          block = true;
        }
      }
      if (!block) {
#pragma unroll
        for (int a = 0; a < NDOF; ++a)
          c += finish_value<OP, DOT, V>(p, n0 * NDOF + a, z[a], ci.w, xs[a], (V)0, dold[a], out[a], dd[a]);
      }
#pragma unroll
      for (int a = 0; a < NDOF; ++a) p.out[(int64_t)ci.x * NDOF + a] = out[a];
      if (t == ci.z) contrib = c;  // a shared node counts once, by its first copy
    }
  }
  if constexpr (DOT || OP == StencilOp::CgQ) {
    const double s = block_sum(contrib);
    if (t == 0) partials[blk] = s;
  }
}

// ------------------------------------------------ 3D scalar stencil, 2.5D tiles
// A block owns a tile of ty x-rows (tx nodes each) of one region and marches nz planes in z.
// The input vector's planes pass through two LDS slots; each thread keeps its 3x3
// neighbourhood of planes z-1, z, z+1 in registers (rotated per plane), so it reads only the
// new plane from LDS, and the plane after next is prefetched from global memory into registers
// while the current plane is computed.  Neighbours outside the region box read 0 from LDS and
// have zero coefficients, so the 27-term sum needs no bounds branches.

// Grid = one block per tile, or (persistent launch) fewer blocks that stride over the tile list.
// SYM: the operator is symmetric and `coef` holds only the upper half of each stencil (offsets
// s = 13..26 of the 27-point order, kSymPts per node, wave-tiled); a lower coupling A(i, i+s),
// s < 13, is the upper coupling A(i+s, i) stored with node i+s at offset 26 - s.  Each thread
// streams its node's 14 couplings once and leaves the ones its neighbours need in LDS: the
// couplings towards z+1 for the next plane, the in-plane ones for this plane.  Only neighbours
// outside the tile (its edge rows, and plane z-1 of the tile's first plane) are read from memory,
// so HBM carries about 14 instead of 27 coefficients per node.
// NT threads per block (the level's tile_threads); tiles hold at most NT nodes.
template <int NT, class V, class C, StencilOp OP, bool DOT, bool SYM>
__global__ __launch_bounds__(NT) void k_stencil3d(LevelView L, const Tile3* __restrict__ tiles, int ntiles,
                                                  const C* __restrict__ coef, const float* __restrict__ centre,
                                                  OpP<V> p, double* __restrict__ partials) {
  constexpr int kT3 = NT;
  constexpr int kT3Plane = tile_plane_cap(NT);
  constexpr int kT3Fetch = (kT3Plane + kT3 - 1) / kT3;
  // Chebyshev steps compute D~^-1 of one-region nodes from the centre coefficient when it is stored
  // in the arithmetic's own type (FP64, or the FP32 copy); the BF16 storage's centre carries the
  // row-sum correction, so it keeps reading the stored reciprocal
  constexpr bool kOwnDiag = std::is_same<V, C>::value && (OP == StencilOp::Cheb || OP == StencilOp::ChebFirst);
  __shared__ V pl[2][kT3Plane];
  // SYM: the previous plane's couplings towards z+1 (9 per tile node) and this plane's in-plane upper
  // couplings (4 per tile node), indexed by the tile-local node = thread index
  __shared__ C sprev[SYM ? 9 : 1][SYM ? kT3 : 1];
  __shared__ C srow[SYM ? 4 : 1][SYM ? kT3 : 1];
  const int t = threadIdx.x;
  double contrib = 0.0;
  // one tile per block: every XCD runs a contiguous run of tiles (xcd_item), so neighbouring
  // tiles' halo rows meet in its L2; persistent grids stride over the tiles
  const bool one = (int)gridDim.x == ntiles;
  for (int it = blockIdx.x; it < ntiles; it += gridDim.x) {
    const Tile3 T = tiles[one ? xcd_item(it, ntiles) : it];
    const RegionGeo R = L.regs[T.region];
    const int W = T.tx + 2, PL = (T.ty + 2) * W;
    const V* __restrict__ xr = p.x + R.off;
    const int ty = t / T.tx, tx = t - ty * T.tx;
    const int x = T.x0 + tx, y = T.y0 + ty;
    const bool active = ty < T.ty && x < R.ex && y < R.ey;
    const int sy = R.ex, sz = R.ex * R.ey;
    V pre[kT3Fetch];
    auto fetch = [&](int zz) {
#pragma unroll
      for (int k = 0; k < kT3Fetch; ++k) {
        const int idx = t + k * kT3;
        V v = (V)0;
        if (idx < PL) {
          const int r = idx / W;
          const int xx = T.x0 + idx - r * W - 1, yy = T.y0 - 1 + r;
          if ((unsigned)zz < (unsigned)R.ez && (unsigned)yy < (unsigned)R.ey && (unsigned)xx < (unsigned)R.ex)
            v = xr[zz * sz + yy * sy + xx];
        }
        pre[k] = v;
      }
    };
    auto store = [&](int slot) {
#pragma unroll
      for (int k = 0; k < kT3Fetch; ++k) {
        const int idx = t + k * kT3;
        if (idx < PL) pl[slot][idx] = pre[k];
      }
    };
    V rm[9], rc[9], rp[9];
    auto readn = [&](int slot, V* r) {
#pragma unroll
      for (int j = 0; j < 9; ++j) {
        const int dx = j % 3 - 1, dy = j / 3 - 1;
        r[j] = pl[slot][(ty + 1 + dy) * W + tx + 1 + dx];
      }
    };
    const int z0 = T.z0, z1 = T.z0 + T.nz;
    // SYM: b and the old direction of this thread's node on the next plane, read a plane ahead
    constexpr bool kPreB = SYM && (OP == StencilOp::Residual || OP == StencilOp::ResidualScaled ||
                                   OP == StencilOp::Cheb || OP == StencilOp::ChebFirst);
    constexpr bool kPreD = SYM && OP == StencilOp::Cheb;
    V nb = (V)0, nd = (V)0;
    auto load_bd = [&](int z2) {
      if (active && z2 < z1) {
        const int64_t g = R.off + (int64_t)z2 * sz + (int64_t)y * sy + x;
        if constexpr (kPreB) nb = p.b[g];
        if constexpr (kPreD) nd = p.out[g];  // u_(k-2), see finish_value
      }
    };
    if constexpr (kPreB) load_bd(z0);
    fetch(z0 - 1);
    store(0);
    fetch(z0);
    store(1);
    __syncthreads();
    if (active) {
      readn(0, rm);
      readn(1, rc);
    }
    __syncthreads();
    fetch(z0 + 1);
    store(0);
    __syncthreads();
    for (int zz = z0; zz < z1; ++zz) {
      const int sp = (zz - z0) & 1;  // slot holding plane zz+1
      const V cb = nb, cd = nd;
      if constexpr (kPreB) load_bd(zz + 1);
      if (active) readn(sp, rp);
      fetch(zz + 2);
      // SYM: own upper couplings u[k] = A(i, i + offset(13 + k)); lower couplings lo[s] = A(i, i +
      // offset(s)) = A(i + offset(s), i), from LDS when the neighbour is a node of this tile (and,
      // for z-1, when this tile computed that plane), else from the neighbour's record in memory.
      V up[SYM ? kSymPts : 1], lo[SYM ? 13 : 1];
      if constexpr (SYM) {
        const int li = zz * sz + y * sy + x;
        const int64_t gi = R.off + li;
        const bool inner = x > 0 && x < R.ex - 1 && y > 0 && y < R.ey - 1 && zz > 0 && zz < R.ez - 1;
        auto nb_ok = [&](int dx, int dy, int dz) {
          return inner || ((unsigned)(x + dx) < (unsigned)R.ex && (unsigned)(y + dy) < (unsigned)R.ey &&
                           (unsigned)(zz + dz) < (unsigned)R.ez);
        };
        auto in_tile = [&](int dx, int dy) {
          return (unsigned)(tx + dx) < (unsigned)T.tx && (unsigned)(ty + dy) < (unsigned)T.ty;
        };
        auto mirror = [&](int s, int dx, int dy, int dz) {  // A(i + offset(s), i) from memory
          return (V)CoefLoad<C>::get(coef + coef_index(gi + dx + dy * sy + dz * sz, 13 - s, kSymPts));
        };
        if (active) {
          const C* __restrict__ cf = coef + coef_index(gi, 0, kSymPts);
#pragma unroll
          for (int k = 0; k < kSymPts; ++k) up[k] = (V)CoefLoad<C>::get(cf + k * kTile);
#pragma unroll
          for (int s = 0; s < 9; ++s) {  // z-1: the neighbour's coupling towards z+1
            const int dx = s % 3 - 1, dy = s / 3 - 1;
            V v = (V)0;
            if (nb_ok(dx, dy, -1)) v = (zz > z0 && in_tile(dx, dy)) ? (V)sprev[8 - s][t + dx + dy * T.tx] : mirror(s, dx, dy, -1);
            lo[s] = v;
          }
#pragma unroll
          for (int k = 1; k < 5; ++k) srow[k - 1][t] = (C)up[k];
        }
        __syncthreads();  // srow visible; every read of sprev done
        if (active) {
#pragma unroll
          for (int k = 5; k < kSymPts; ++k) sprev[k - 5][t] = (C)up[k];
#pragma unroll
          for (int s = 9; s < 13; ++s) {  // in-plane lower couplings
            int dx, dy, dz;
            stencil_offset<27>(s, dx, dy, dz);
            V v = (V)0;
            if (nb_ok(dx, dy, 0)) v = in_tile(dx, dy) ? (V)srow[12 - s][t + dx + dy * T.tx] : mirror(s, dx, dy, 0);
            lo[s] = v;
          }
        }
      }
      if (active) {
        const int li = zz * sz + y * sy + x;
        const int64_t gi = R.off + li;
        V acc = (V)0, ctr = (V)0;  // ctr: centre coefficient (the diagonal of a one-region node)
        if constexpr (SYM) {
          // stencil order, one rounding each (as k_stencil_table sums them)
#pragma unroll
          for (int s = 0; s < 27; ++s) {
            const int j = s % 9;
            acc = fma(s < 13 ? lo[s] : up[s - 13], s < 9 ? rm[j] : (s < 18 ? rc[j] : rp[j]), acc);
          }
          ctr = up[0];
        } else {
          const C* __restrict__ cf = coef + coef_index(gi, 0, 27);
#pragma unroll
          for (int s = 0; s < 27; ++s) {
            const int j = s % 9, dz = s / 9 - 1;
            const V v = dz < 0 ? rm[j] : (dz == 0 ? rc[j] : rp[j]);
            const V cv = (V)coefv<27, 1, C>(cf, centre, gi, s, 0, 0);
            if (s == 13) ctr = cv;
            acc += cv * v;
          }
        }
        const bool edge = x == 0 || x == R.ex - 1 || y == 0 || y == R.ey - 1 || zz == 0 || zz == R.ez - 1;
        if (edge && is_shared(L, R, x, y, zz)) {  // finished by k_iface
          if constexpr (kPreD) write_partial<OP, V>(p, gi, acc, rc[4], cd);
          else write_partial<OP, V>(p, gi, acc, rc[4], OP == StencilOp::Cheb ? p.out[gi] : (V)0);
        } else if constexpr (kPreB) contrib += finish_pre<OP, DOT, V, kOwnDiag>(p, gi, acc, 1, rc[4], ctr, cb, cd);
        else contrib += finish<OP, DOT, V, kOwnDiag>(p, gi, acc, 1, rc[4], ctr);
      }
      store(sp ^ 1);  // plane zz+2 replaces plane zz
#pragma unroll
      for (int j = 0; j < 9; ++j) {
        rm[j] = rc[j];
        rc[j] = rp[j];
      }
      __syncthreads();
    }
  }
  if constexpr (DOT || OP == StencilOp::CgQ) {
    double v = contrib;
    for (int o = 32; o > 0; o >>= 1) v += __shfl_down(v, o, 64);
    __shared__ double sm[kT3 / 64];
    if ((t & 63) == 0) sm[t >> 6] = v;
    __syncthreads();
    if (t == 0) {
      double s = 0.0;
      for (int i = 0; i < kT3 / 64; ++i) s += sm[i];
      // one tile per block: the tile's slot, as without the mapping
      partials[one ? xcd_item((int)blockIdx.x, ntiles) : (int)blockIdx.x] = s;
    }
  }
}

// ------------------------------------------------------- region-table tiles

// Whole-region tiles of a region served by its class tables: ty full x-rows, nz planes.  The lanes
// of the rows' inner nodes (x in [2, ex - 2)) come first, padded to whole wavefronts, then the rows'
// four x-face nodes.  A node's couplings are its class's (scalar loads from the region's table): a
// wavefront takes the classes of its nodes one after the other, so one whose nodes share a class
// (every inner wavefront away from the y-faces) runs one pass.  No coupling is read per node.  The
// input vector's planes, whole rows with their halo, pass through two LDS slots; each plane is
// fetched four planes ahead into registers and b and u_(k-2) two planes ahead, so that two planes'
// loads are in flight while one is computed, and each plane read adds its products to the running
// sums of the three nodes it neighbours in z.  The kernel is held to 80 VGPRs (six waves per SIMD,
// three 8-wave blocks per CU), at the cost of one spilled register in the Chebyshev step; the
// variant that also sums (b, u_out) keeps five waves, where it needs no spill.  FP32 vectors (the
// low-precision cycle, with its own tables) fit eight waves: on 113M rows in 256 uneven regions a
// Chebyshev step takes 546 us, 3.3 TB/s on its 16 B a row, where streaming 14 couplings a row took
// 2081 us, and the FP64 CG product of that solve 575 instead of 3649 us.  Blocks
// are mapped to tiles so that every XCD runs a contiguous run of tiles (xcd_item) and neighbouring
// tiles share their halo rows through its L2.  Every node sums its 27 products in stencil order with
// one rounding each, as k_stencil3d does, so the results are those of streaming every coupling bit
// for bit.
template <class V, StencilOp OP, bool DOT, bool DINV>
__global__ __launch_bounds__(kTableThreads) __attribute__((amdgpu_waves_per_eu(sizeof(V) == 4 ? 8 : (DOT ? 5 : 6)))) void k_stencil_table(
    LevelView L, const Tile3* __restrict__ tiles, const V* __restrict__ table, const V* __restrict__ cdinv, OpP<V> p,
    double* __restrict__ partials) {
  constexpr int NT = kTableThreads;
  constexpr int kPlane = 2 * NT;  // a tile's rows with their halo: two loads per lane (make_split)
  constexpr int kFetch = 2;
  constexpr bool kPreB = OP == StencilOp::Residual || OP == StencilOp::ResidualScaled || OP == StencilOp::Cheb ||
                         OP == StencilOp::ChebFirst;
  constexpr bool kPreD = OP == StencilOp::Cheb;
  constexpr int kOwn = DINV ? kOwnDinv : kOwnCentre;
  constexpr int kXCols = 20;  // classes of the x-face nodes in a plane: five y classes, four x classes
  __shared__ V pl[2][kPlane];
  __shared__ V xt[5][kClassPts][kXCols];  // the x-face lanes' couplings by z class
  __shared__ V xd[DINV ? 5 : 1][kXCols];  // and their D~^-1
  const Tile3 T = tiles[xcd_item((int)blockIdx.x, (int)gridDim.x)];
  const RegionGeo R = L.regs[T.region];
  const V* __restrict__ tab = table + (int64_t)T.region * kClasses * kClassPts;
  const V* __restrict__ dtab = DINV ? cdinv + (int64_t)T.region * kClasses : nullptr;
  const int t = threadIdx.x;
  // lane -> (row, x): inner-x lanes, padded to a wavefront boundary, then x-face lanes
  const int dxw = R.ex - 4, ndl = T.ty * dxw, pad = (ndl + 63) & ~63;
  int row = 0, x = 0;
  bool active = false;
  if (t < ndl) {
    row = t / dxw;
    x = 2 + t - row * dxw;
    active = true;
  } else if (t >= pad && t < pad + 4 * T.ty) {
    const int u = t - pad;
    row = u >> 2;
    x = (u & 3) < 2 ? (u & 3) : R.ex - 4 + (u & 3);
    active = true;
  }
  const int y = T.y0 + row;
  const int cxy = axis_class(y, R.ey) * 5 + axis_class(x, R.ex);
  const int W = R.ex + 2, PL = (T.ty + 2) * W;
  const int sy = R.ex, sz = R.ex * R.ey;
  const V* __restrict__ xr = p.x + R.off;
  // Loads are issued unconditionally (out-of-range positions read a valid element and are zeroed
  // when stored), so that the compiler counts the loads in flight exactly and waits only for the
  // plane it needs.
  auto fetch = [&](int zz, V(&pre)[kFetch]) {
    const int zc = min(max(zz, 0), R.ez - 1);
#pragma unroll
    for (int k = 0; k < kFetch; ++k) {
      const int idx = min(t + k * NT, PL - 1);
      const int r = idx / W;
      const int xx = min(max(idx - r * W - 1, 0), R.ex - 1), yy = min(max(T.y0 - 1 + r, 0), R.ey - 1);
      pre[k] = xr[(int64_t)zc * sz + (int64_t)yy * sy + xx];
    }
  };
  auto store = [&](int slot, int zz, const V(&pre)[kFetch]) {
#pragma unroll
    for (int k = 0; k < kFetch; ++k) {
      const int idx = t + k * NT;
      if (idx < PL) {
        const int r = idx / W;
        const int xx = idx - r * W - 1, yy = T.y0 - 1 + r;
        const bool in = (unsigned)zz < (unsigned)R.ez && (unsigned)yy < (unsigned)R.ey && (unsigned)xx < (unsigned)R.ex;
        pl[slot][idx] = in ? pre[k] : (V)0;
      }
    }
  };
  V v9[9];  // this lane's 3 x 3 neighbourhood on the plane read last
  auto readn = [&](int slot) {
#pragma unroll
    for (int j = 0; j < 9; ++j) v9[j] = pl[slot][(row + j / 3) * W + x + j % 3];
  };
  const int z0 = T.z0, z1 = T.z0 + T.nz;
  auto load_bd = [&](int z2, V& b2, V& d2) {  // inactive lanes and planes past the tile: a valid node
    const int64_t g = R.off + (int64_t)min(z2, z1 - 1) * sz + (int64_t)y * sy + x;
    if constexpr (kPreB) b2 = p.b[g];
    if constexpr (kPreD) d2 = p.out[g];  // u_(k-2), see finish_value
  };
  for (int e = t; e < 5 * kClassPts * kXCols; e += NT) {  // couplings of the x-face classes
    const int u = e % kXCols, s2 = e / kXCols % kClassPts, cz = e / (kXCols * kClassPts);
    const int cx = (u & 3) < 2 ? (u & 3) : (u & 3) + 1;
    xt[cz][s2][u] = tab[((cz * 5 + (u >> 2)) * 5 + cx) * kClassPts + s2];
    if (DINV && s2 == 13) xd[cz][u] = dtab[(cz * 5 + (u >> 2)) * 5 + cx];
  }
  // Running sums: once plane q has been added, a0 is node q - 1's sum, a1 node q's and a2 node
  // q + 1's.  A plane adds its nine values to the three nodes it neighbours in z (as their plane
  // z + 1, z and z - 1), so each node adds its 27 products in stencil order with one rounding each,
  // and only the plane read last is held in registers.
  V a0 = (V)0, a1 = (V)0, a2 = (V)0, ctr = (V)0, xprev = (V)0;
  auto czc = [&](int z) { return min(max(axis_class(z, R.ez), 0), 4); };
  auto add_plane = [&](int q) {
    a2 = (V)0;
    if (t >= pad) {
      // the x-face wavefronts (four classes a row): each lane reads its class's couplings from
      // the block's copy in LDS, nine at a time (the empty asm keeps the chunks' reads apart)
      const int u = axis_class(y, R.ey) * 4 + ((t - pad) & 3);
      auto chunk = [&](const V* __restrict__ xc, V& acc) {
        V cf[9];
#pragma unroll
        for (int j = 0; j < 9; ++j) cf[j] = xc[j * kXCols];
#pragma unroll
        for (int j = 0; j < 9; ++j) acc = fma(cf[j], v9[j], acc);
        __asm__ volatile("" ::: "memory");
      };
      chunk(&xt[czc(q - 1)][18][u], a0);
      chunk(&xt[czc(q)][9][u], a1);
      chunk(&xt[czc(q + 1)][0][u], a2);
      ctr = DINV ? xd[czc(q - 1)][u] : xt[czc(q - 1)][13][u];
    } else {
      // the classes of this wavefront's nodes, one after the other (the mask of lanes left and the
      // leading lane are wavefront-uniform, so every pass reads its class afresh)
      uint64_t left = __builtin_amdgcn_ballot_w64(true);
      while (left) {
        const int c = __builtin_amdgcn_readlane(cxy, (int)__builtin_ctzll(left));
        // the three classes' table offsets, in scalar registers the compiler cannot trade for
        // per-lane values below, so that the table is read with scalar loads
        int o0 = __builtin_amdgcn_readfirstlane((czc(q - 1) * 25 + c) * kClassPts);
        int o1 = __builtin_amdgcn_readfirstlane((czc(q) * 25 + c) * kClassPts);
        int o2 = __builtin_amdgcn_readfirstlane((czc(q + 1) * 25 + c) * kClassPts);
        __asm__ volatile("" : "+s"(o0), "+s"(o1), "+s"(o2));
        const bool mine = cxy == c;
        if (mine) {
          const V* __restrict__ t0 = tab + o0;
          const V* __restrict__ t1 = tab + o1;
          const V* __restrict__ t2 = tab + o2;
#pragma unroll
          for (int j = 0; j < 9; ++j) a0 = fma(t0[18 + j], v9[j], a0);
#pragma unroll
          for (int j = 0; j < 9; ++j) a1 = fma(t1[9 + j], v9[j], a1);
#pragma unroll
          for (int j = 0; j < 9; ++j) a2 = fma(t2[j], v9[j], a2);
          ctr = DINV ? dtab[o0 / kClassPts] : t0[13];
        }
        left &= ~__builtin_amdgcn_ballot_w64(mine);
      }
    }
  };
  auto shift = [&]() {
    a0 = a1;
    a1 = a2;
    xprev = v9[4];
  };
  V preA[kFetch], preB[kFetch];
  V nbA = (V)0, ndA = (V)0, nbB = (V)0, ndB = (V)0;
  load_bd(z0, nbA, ndA);
  load_bd(z0 + 1, nbB, ndB);
  fetch(z0 - 1, preA);
  fetch(z0, preB);
  store(0, z0 - 1, preA);
  store(1, z0, preB);
  __syncthreads();
  if (active) {  // planes z0 - 1 and z0: the first two thirds of node z0, the first of z0 + 1
    readn(0);
    add_plane(z0 - 1);
    shift();
    readn(1);
    add_plane(z0);
    shift();
  }
  __syncthreads();
  fetch(z0 + 1, preA);
  store(0, z0 + 1, preA);
  fetch(z0 + 2, preA);
  fetch(z0 + 3, preB);
  __syncthreads();
  double contrib = 0.0;
  // one plane: plane zz + 1 from LDS completes node zz; plane zz + 2 goes to LDS from the
  // registers that fetched it two planes ago, which then fetch plane zz + 4 (past the tile's last
  // plane it only keeps the loads in step: see the loop below)
  auto plane = [&](int zz, V(&pre)[kFetch], V& b2, V& d2) {
    const int sp = (zz - z0) & 1;  // slot holding plane zz + 1
    const bool work = active && zz < z1;
    if (work) readn(sp);
    if (zz + 2 <= z1) store(sp ^ 1, zz + 2, pre);  // plane zz + 2 replaces plane zz
    fetch(zz + 4, pre);
    const V cb = b2, cd = d2;
    load_bd(zz + 2, b2, d2);
    if (work) {
      add_plane(zz + 1);
      const int64_t gi = R.off + (int64_t)zz * sz + (int64_t)y * sy + x;
      const bool edge = x == 0 || x == R.ex - 1 || y == 0 || y == R.ey - 1 || zz == 0 || zz == R.ez - 1;
      if (edge && is_shared(L, R, x, y, zz)) write_partial<OP, V>(p, gi, a0, xprev, cd);  // finished by k_iface
      else if constexpr (kPreB) contrib += finish_pre<OP, DOT, V, kOwn>(p, gi, a0, 1, xprev, ctr, cb, cd);
      else contrib += finish<OP, DOT, V, kOwn>(p, gi, a0, 1, xprev, ctr);
      shift();
    }
    __syncthreads();
  };
  // Both halves run on every pass, also past the last plane, so that every pass issues the same
  // loads and the compiler's count of loads in flight stays exact around the loop.
  for (int zz = z0; zz < z1; zz += 2) {
    plane(zz, preA, nbA, ndA);
    plane(zz + 1, preB, nbB, ndB);
  }
  if constexpr (DOT || OP == StencilOp::CgQ) {
    double v = contrib;
    for (int o = 32; o > 0; o >>= 1) v += __shfl_down(v, o, 64);
    __shared__ double sm[NT / 64];
    if ((t & 63) == 0) sm[t >> 6] = v;
    __syncthreads();
    if (t == 0) {
      double s = 0.0;
      for (int i = 0; i < NT / 64; ++i) s += sm[i];
      partials[blockIdx.x] = s;
    }
  }
}

// ------------------------------------------------- region-table tiles, 3 dofs

// k_stencil_table for 3-dof levels: 3 x 3 coupling blocks, 243 products a node, from the region's
// table by scalar loads.  A tile is a few whole rows without their x-face nodes, or (pad 1) the four
// x-face columns of up to 64 rows, a wavefront a column, so that in either a wavefront's nodes are
// almost all of one class.  Planes of three-vectors pass through two LDS slots as there, and each plane
// read adds its products to the running sums of the three nodes it neighbours in z; every node's
// sums are k_stencil's, product for product, so the results are bit for bit those of node blocks.
// 27 regions of 55^3 (4.5M nodes): CG product 405 us on node blocks, 272 here, a Chebyshev step 490 and
// 364 (its inner product is a pass of its own, 22 us: in the step it spilled 30 registers and took 446
// in all), an FP32 Chebyshev step 177 (streaming BF16 blocks 478).  A step is
// bound by the latency between planes: 128 to 168 VGPRs leave twelve wavefronts a CU, whose 31 scalar
// loads and one plane's memory latency a step the 243 products (1,000 cycles) only half cover.  Taking
// the x-face columns' classes one after the other by scalar loads instead of from LDS cost 440 us (their
// 20 classes of 2 KB do not fit the scalar cache), one plane in flight instead of two 10% more.
template <class V, StencilOp OP>
__global__ __launch_bounds__(kTable3Threads) __attribute__((amdgpu_waves_per_eu(sizeof(V) == 4 ? 4 : 3))) void k_stencil_table3(
                                                                   LevelView L, const Tile3* __restrict__ tiles,
                                                                   const V* __restrict__ table, OpP<V> p,
                                                                   double* __restrict__ partials) {
  constexpr int NT = kTable3Threads, kFetch = kTable3Fetch;
  constexpr bool kPreB = OP == StencilOp::Residual || OP == StencilOp::ResidualScaled || OP == StencilOp::Cheb ||
                         OP == StencilOp::ChebFirst;
  constexpr bool kPreD = OP == StencilOp::Cheb;
  constexpr bool kOwn = std::is_same<V, double>::value;  // D~^-1 of a one-region row as 1 / its centre entry
  __shared__ V pl[2][kFetch * NT];
  // x-face tiles: the couplings of the plane's 20 classes (five along y, four along x), the part of each
  // stencil plane from the z class of the node that it belongs to
  constexpr int kCols = 20, kRow = kClassPts * 9;
  __shared__ V ft[kCols * kRow];
  const Tile3 T = tiles[xcd_item((int)blockIdx.x, (int)gridDim.x)];
  const RegionGeo R = L.regs[T.region];
  // the table in the constant address space: no store of this kernel reaches it, so uniform reads are
  // scalar loads (the compiler does not prove that by itself across a loop with this many accesses)
  using Tab = const V __attribute__((address_space(4)))*;
  const Tab tab = (Tab)(uintptr_t)(table + (int64_t)T.region * kClasses * kClassPts * 9);
  const int t = threadIdx.x;
  const bool face = T.pad != 0;
  int row = 0, x = 2, col = 3;
  bool active = false;
  if (face) {
    const int w = t >> 6, l = t & 63;
    if (w < 4 && l < T.ty) {
      row = l;
      x = w < 2 ? w : R.ex - 4 + w;
      col = w < 2 ? w + 1 : w + 3;
      active = true;
    }
  } else if (t < T.ty * (R.ex - 4)) {
    row = t / (R.ex - 4);
    x = 2 + t - row * (R.ex - 4);
    col = x + 1;
    active = true;
  }
  const int y = T.y0 + row;
  const int cxy = axis_class(y, R.ey) * 5 + axis_class(x, R.ex);
  // staged columns: the whole row with its halo, or x = -1 .. 2 and ex - 3 .. ex
  const int WC = 3 * (face ? 8 : R.ex + 2), PL = (T.ty + 2) * WC;
  const int sy = R.ex, sz = R.ex * R.ey;
  const V* __restrict__ xr = p.x + R.off * 3;
  int off[kFetch];
  unsigned inside = 0;
#pragma unroll
  for (int k = 0; k < kFetch; ++k) {
    const int idx = min(t + k * NT, PL - 1), r = idx / WC, c = idx - r * WC, q = c / 3;
    const int xx = face && q >= 4 ? R.ex - 7 + q : q - 1, yy = T.y0 - 1 + r;
    if ((unsigned)yy < (unsigned)R.ey && (unsigned)xx < (unsigned)R.ex) inside |= 1u << k;
    off[k] = (min(max(yy, 0), R.ey - 1) * sy + min(max(xx, 0), R.ex - 1)) * 3 + c - 3 * q;
  }
  auto fetch = [&](int zz, V(&pre)[kFetch]) {
    const V* __restrict__ xz = xr + (int64_t)min(max(zz, 0), R.ez - 1) * sz * 3;
#pragma unroll
    for (int k = 0; k < kFetch; ++k) pre[k] = xz[off[k]];
  };
  auto store = [&](int slot, int zz, const V(&pre)[kFetch]) {
    const bool zin = (unsigned)zz < (unsigned)R.ez;
#pragma unroll
    for (int k = 0; k < kFetch; ++k) {
      const int idx = t + k * NT;
      if (idx < PL) pl[slot][idx] = zin && (inside >> k & 1u) ? pre[k] : (V)0;
    }
  };
  V v[27];  // this lane's 3 x 3 neighbours' three-vectors on the plane read last
  auto readn = [&](int slot) __attribute__((always_inline)) {
#pragma unroll
    for (int j = 0; j < 9; ++j)
#pragma unroll
      for (int b = 0; b < 3; ++b) v[j * 3 + b] = pl[slot][(row + j / 3) * WC + (col - 1 + j % 3) * 3 + b];
  };
  const int z0 = T.z0, z1 = T.z0 + T.nz;
  auto load_bd = [&](int z2, V(&b2)[3], V(&d2)[3]) {  // inactive lanes and planes past the tile: a valid node
    const int64_t g = (R.off + (int64_t)min(z2, z1 - 1) * sz + (int64_t)y * sy + x) * 3;
#pragma unroll
    for (int a = 0; a < 3; ++a) {
      if constexpr (kPreB) b2[a] = p.b[g + a];
      if constexpr (kPreD) d2[a] = p.out[g + a];  // u_(k-2), see finish_value
    }
  };
  // running sums as in k_stencil_table
  V a0[3] = {}, a1[3] = {}, a2[3] = {}, ctr[3] = {}, xprev[3] = {};
  auto czc = [&](int z) { return min(max(axis_class(z, R.ez), 0), 4); };
  int key = -1;  // z classes of the couplings in ft
  auto load_faces = [&](int q) {  // every thread of an x-face tile, before the plane's products
    const int c0 = czc(q - 1), c1 = czc(q), c2 = czc(q + 1), want = (c0 * 5 + c1) * 5 + c2;
    if (want == key) return;
    key = want;
    for (int e = t; e < kCols * kRow; e += NT) {
      const int u = e / kRow, i = e - u * kRow, cx = (u & 3) < 2 ? (u & 3) : (u & 3) + 1;
      const int cz = i < 81 ? c2 : (i < 162 ? c1 : c0);
      ft[e] = tab[((cz * 5 + (u >> 2)) * 5 + cx) * kRow + i];
    }
    __syncthreads();
  };
  const int fu = (axis_class(y, R.ey) * 4 + min(t >> 6, 3)) * kRow;
  auto add_plane = [&](int q) __attribute__((always_inline)) {
#pragma unroll
    for (int a = 0; a < 3; ++a) a2[a] = (V)0;
    if (face) {  // each lane reads its class's couplings, one row of a block at a time
      auto part = [&](int s0, V(&acc)[3]) __attribute__((always_inline)) {
#pragma unroll
        for (int j = 0; j < 9; ++j) {
          V cf[9];
#pragma unroll
          for (int e = 0; e < 9; ++e) cf[e] = ft[fu + (s0 + j) * 9 + e];
#pragma unroll
          for (int a = 0; a < 3; ++a)
#pragma unroll
            for (int b = 0; b < 3; ++b) acc[a] = fma(cf[a * 3 + b], v[j * 3 + b], acc[a]);
          if (j % 2) __asm__ volatile("" ::: "memory");
        }
      };
      part(18, a0);
      part(9, a1);
      part(0, a2);
      if constexpr (kOwn) {  // (of the node that this plane completes: class czc(q - 1))
        const int cz = czc(q - 1) * 25 + cxy;
#pragma unroll
        for (int a = 0; a < 3; ++a) ctr[a] = tab[cz * kRow + 13 * 9 + a * 4];
      }
      return;
    }
    uint64_t left = __builtin_amdgcn_ballot_w64(true);
    while (left) {
      const int c = __builtin_amdgcn_readlane(cxy, (int)__builtin_ctzll(left));
      int o0 = __builtin_amdgcn_readfirstlane((czc(q - 1) * 25 + c) * kClassPts * 9);
      int o1 = __builtin_amdgcn_readfirstlane((czc(q) * 25 + c) * kClassPts * 9);
      int o2 = __builtin_amdgcn_readfirstlane((czc(q + 1) * 25 + c) * kClassPts * 9);
      __asm__ volatile("" : "+s"(o0), "+s"(o1), "+s"(o2));
      const bool mine = cxy == c;
      if (mine) {
        const Tab t0 = tab + o0 + 18 * 9, t1 = tab + o1 + 9 * 9, t2 = tab + o2;
#pragma unroll
        for (int j = 0; j < 9; ++j)
#pragma unroll
          for (int a = 0; a < 3; ++a)
#pragma unroll
            for (int b = 0; b < 3; ++b) a0[a] = fma(t0[(j * 3 + a) * 3 + b], v[j * 3 + b], a0[a]);
#pragma unroll
        for (int j = 0; j < 9; ++j)
#pragma unroll
          for (int a = 0; a < 3; ++a)
#pragma unroll
            for (int b = 0; b < 3; ++b) a1[a] = fma(t1[(j * 3 + a) * 3 + b], v[j * 3 + b], a1[a]);
#pragma unroll
        for (int j = 0; j < 9; ++j)
#pragma unroll
          for (int a = 0; a < 3; ++a)
#pragma unroll
            for (int b = 0; b < 3; ++b) a2[a] = fma(t2[(j * 3 + a) * 3 + b], v[j * 3 + b], a2[a]);
        if constexpr (kOwn) {
#pragma unroll
          for (int a = 0; a < 3; ++a) ctr[a] = tab[o0 + 13 * 9 + a * 4];
        }
      }
      left &= ~__builtin_amdgcn_ballot_w64(mine);
    }
  };
  auto shift = [&]() {
#pragma unroll
    for (int a = 0; a < 3; ++a) {
      a0[a] = a1[a];
      a1[a] = a2[a];
      xprev[a] = v[12 + a];
    }
  };
  V preA[kFetch], preB[kFetch];
  fetch(z0 - 1, preA);
  fetch(z0, preB);
  store(0, z0 - 1, preA);
  store(1, z0, preB);
  fetch(z0 + 1, preA);
  fetch(z0 + 2, preB);
  __syncthreads();
  if (face) load_faces(z0 - 1);
  if (active) {
    readn(0);
    add_plane(z0 - 1);
    shift();
  }
  __syncthreads();
  if (face) load_faces(z0);
  if (active) {
    readn(1);
    add_plane(z0);
    shift();
  }
  __syncthreads();
  store(0, z0 + 1, preA);
  fetch(z0 + 3, preA);
  __syncthreads();
  double contrib = 0.0;
  auto plane = [&](int zz, V(&pre)[kFetch]) __attribute__((always_inline)) {
    const int sp = (zz - z0) & 1;  // slot holding plane zz + 1
    const bool work = active && zz < z1;
    if (face) load_faces(zz + 1);
    if (work) readn(sp);
    if (zz + 2 <= z1) store(sp ^ 1, zz + 2, pre);  // plane zz + 2 replaces plane zz
    V cb[3] = {}, cd[3] = {};
    load_bd(zz, cb, cd);  // used after the plane's 243 products; issued before the fetch, so not behind it
    fetch(zz + 4, pre);
    if (work) {
      add_plane(zz + 1);
      const int64_t node = R.off + (int64_t)zz * sz + (int64_t)y * sy + x;
      const bool edge = x == 0 || x == R.ex - 1 || y == 0 || y == R.ey - 1 || zz == 0 || zz == R.ez - 1;
      if (edge && is_shared(L, R, x, y, zz)) {  // finished by k_iface
#pragma unroll
        for (int a = 0; a < 3; ++a) write_partial<OP, V>(p, node * 3 + a, a0[a], xprev[a], cd[a]);
      } else {
        bool block = false;
        if constexpr (OP == StencilOp::Cheb || OP == StencilOp::ChebFirst) {
          if (p.dinv9) {
            V dold[3], out[3], dd[3];
#pragma unroll
            for (int a = 0; a < 3; ++a)
              dold[a] = OP == StencilOp::Cheb ? prev_correction(p, xprev[a], cd[a]) : xprev[a];
            contrib += finish_block3_value<OP, false, V>(p, node, a0, xprev, dold, out, dd);
#pragma unroll
            for (int a = 0; a < 3; ++a) p.out[node * 3 + a] = out[a];
            block = true;
          }
        }
        if (!block) {
#pragma unroll
          for (int a = 0; a < 3; ++a) {
            if constexpr (kPreB)
              contrib += finish_pre<OP, false, V, kOwn>(p, node * 3 + a, a0[a], 1, xprev[a], ctr[a], cb[a], cd[a]);
            else
              contrib += finish<OP, false, V, kOwn>(p, node * 3 + a, a0[a], 1, xprev[a], ctr[a]);
          }
        }
      }
      shift();
    }
    __syncthreads();
  };
  // both halves run on every pass, see k_stencil_table
  for (int zz = z0; zz < z1; zz += 2) {
    plane(zz, preB);
    plane(zz + 1, preA);
  }
  if constexpr (OP == StencilOp::CgQ) {
    double s1 = contrib;
    for (int o = 32; o > 0; o >>= 1) s1 += __shfl_down(s1, o, 64);
    __shared__ double sm[NT / 64];
    if ((t & 63) == 0) sm[t >> 6] = s1;
    __syncthreads();
    if (t == 0) {
      double s = 0.0;
      for (int i = 0; i < NT / 64; ++i) s += sm[i];
      partials[blockIdx.x] = s;
    }
  }
}

// ------------------------------------------------------- element tiles

// Whole-row tiles of regions of the finest level whose operator was assembled from element-wise
// diffusion coefficients (FP64).  A node's 27 couplings are sums over its eight elements of element
// matrix entry times coefficient: they are assembled in registers, in the order and with the roundings
// of k_assemble_q1, from one coefficient an element (8 B a node) instead of being streamed (112 B a
// node); a mirrored coupling is the same sum seen from the neighbour, element for element (the element
// matrix is symmetric bit for bit), so every coupling is the one k_stencil3d reads, bit for bit.  On 64
// regions of 82^3 a Chebyshev step takes 430 us, 3.3 TB/s on its 40 B a row, where k_stencil3d takes
// 1170 us.  What bounds it now is the 91 FMAs a node and their uniform operands: with the element
// matrix's 64 entries read again for every plane by scalar loads a step took 540 us, with the 36
// entries on and above the diagonal, which nearly fit the scalar registers, 430.  The layout follows
// k_stencil_table: node planes and element layers pass through two LDS slots each, fetched four ahead,
// and each plane adds its products to the running sums of the three nodes it neighbours in z.
// Elements outside the region count 0.  Couplings to Dirichlet nodes are dropped by taking those nodes'
// values as 0; a Dirichlet row is its stored centre coupling times its own value.
template <StencilOp OP, bool DOT>
__global__ __launch_bounds__(kTableThreads) __attribute__((amdgpu_waves_per_eu(4))) void k_stencil_elem(
    LevelView L, const Tile3* __restrict__ tiles, const double* __restrict__ elem, Kmat K,
    const double* __restrict__ sym, OpP<double> p, double* __restrict__ partials) {
  constexpr int NT = kTableThreads;
  constexpr int kPlane = 2 * NT;  // a tile's nodes with their halo, and its elements: two loads per lane
  constexpr bool kPreB = OP == StencilOp::Residual || OP == StencilOp::ResidualScaled || OP == StencilOp::Cheb ||
                         OP == StencilOp::ChebFirst;
  constexpr bool kPreD = OP == StencilOp::Cheb;
  __shared__ double pl[2][kPlane], el[2][kPlane];
  const Tile3 T = tiles[xcd_item((int)blockIdx.x, (int)gridDim.x)];
  const RegionGeo R = L.regs[T.region];
  const int t = threadIdx.x;
  const int row = t / T.tx, x = t - row * T.tx, y = T.y0 + row;
  const bool active = row < T.ty;
  const int W = R.ex + 2, PL = (T.ty + 2) * W, WE = R.ex + 1, PE = (T.ty + 1) * WE;
  const int sy = R.ex, sz = R.ex * R.ey;
  const double* __restrict__ xr = p.x + R.off;
  const int64_t esy = L.cx - 1, esz = (int64_t)(L.cx - 1) * (L.cy - 1);
  const double* __restrict__ er = elem + R.oz * esz + R.oy * esy + R.ox;
  // this lane's two node and two element positions of a plane: offset of a valid one, and whether it counts
  int noff[2], eoff[2];
  bool nin[2], ein[2];
#pragma unroll
  for (int k = 0; k < 2; ++k) {
    int idx = min(t + k * NT, PL - 1), r = idx / W;
    int xx = idx - r * W - 1, yy = T.y0 - 1 + r;
    nin[k] = (unsigned)yy < (unsigned)R.ey && (unsigned)xx < (unsigned)R.ex;
    if (nin[k])  // Dirichlet nodes on the x and y faces
      nin[k] = !(((L.mask & 1u) && R.ox + xx == 0) || ((L.mask & 2u) && R.ox + xx == L.cx - 1) ||
                 ((L.mask & 4u) && R.oy + yy == 0) || ((L.mask & 8u) && R.oy + yy == L.cy - 1));
    noff[k] = min(max(yy, 0), R.ey - 1) * sy + min(max(xx, 0), R.ex - 1);
    idx = min(t + k * NT, PE - 1), r = idx / WE;
    xx = idx - r * WE - 1, yy = T.y0 - 1 + r;
    ein[k] = (unsigned)yy < (unsigned)(R.ey - 1) && (unsigned)xx < (unsigned)(R.ex - 1);
    eoff[k] = min(max(yy, 0), R.ey - 2) * (int)esy + min(max(xx, 0), R.ex - 2);
  }
  auto fetch = [&](int zz, double(&pre)[4]) {  // nodes of plane zz, elements between planes zz and zz + 1
    const double* __restrict__ xz = xr + (int64_t)min(max(zz, 0), R.ez - 1) * sz;
    const double* __restrict__ ez = er + (int64_t)min(max(zz, 0), R.ez - 2) * esz;
#pragma unroll
    for (int k = 0; k < 2; ++k) {
      pre[k] = xz[noff[k]];
      pre[2 + k] = ez[eoff[k]];
    }
  };
  auto store = [&](int slot, int zz, const double(&pre)[4]) {
    const int gz = R.oz + zz;
    const bool zn = (unsigned)zz < (unsigned)R.ez && !(((L.mask & 16u) && gz == 0) || ((L.mask & 32u) && gz == L.cz - 1));
    const bool ze = (unsigned)zz < (unsigned)(R.ez - 1);
#pragma unroll
    for (int k = 0; k < 2; ++k) {
      const int idx = t + k * NT;
      if (idx < PL) pl[slot][idx] = nin[k] && zn ? pre[k] : 0.0;
      if (idx < PE) el[slot][idx] = ein[k] && ze ? pre[2 + k] : 0.0;
    }
  };
  double v9[9], cm[4], cp[4];  // plane q's 3 x 3 nodes; elements (x - ax, y - ay) below and above it, ax + 2 ay
  auto readn = [&](int slot) {
#pragma unroll
    for (int j = 0; j < 9; ++j) v9[j] = pl[slot][(row + j / 3) * W + x + j % 3];
#pragma unroll
    for (int a = 0; a < 4; ++a) {
      cm[a] = cp[a];
      cp[a] = el[slot][(row + 1 - (a >> 1)) * WE + x + 1 - (a & 1)];
    }
  };
  const int z0 = T.z0, z1 = T.z0 + T.nz;
  auto load_bd = [&](int z2, double& b2, double& d2) {  // inactive lanes and planes past the tile: a valid node
    const int64_t g = R.off + (int64_t)min(z2, z1 - 1) * sz + (int64_t)(active ? y * sy + x : 0);
    if constexpr (kPreB) b2 = p.b[g];
    if constexpr (kPreD) d2 = p.out[g];  // u_(k-2), see finish_value
  };
  // running sums as in k_stencil_table: once plane q has been added, a0 is node q - 1's sum, a1 node
  // q's, a2 node q + 1's; c0 and c1 the centre couplings of nodes q - 1 and q
  double a0 = 0.0, a1 = 0.0, a2 = 0.0, c0 = 0.0, c1 = 0.0, xprev = 0.0;
  double w[9];
  // the element matrix is symmetric bit for bit: its 36 entries on and above the diagonal
  auto ks = [&](int a, int b) { return K.k[min(a, b) * 8 + max(a, b)]; };
  // w[j] += sum over corner roles a of the node (its element c[a & 3]) and b of the neighbour, both
  // four corners of a z layer: the couplings of one stencil plane
  auto couple = [&](const double(&c)[4], int a0c, int b0c) {
#pragma unroll
    for (int a = 0; a < 4; ++a)
#pragma unroll
      for (int b = 0; b < 4; ++b) {
        const int j = ((b >> 1) - (a >> 1) + 1) * 3 + (b & 1) - (a & 1) + 1;
        w[j] = fma(ks(a0c + a, b0c + b), c[a], w[j]);
      }
  };
  auto clear = [&]() {
#pragma unroll
    for (int j = 0; j < 9; ++j) w[j] = 0.0;
  };
  auto add_plane = [&]() {
    clear();
    couple(cm, 0, 4);  // node q - 1 (bottom corners), plane above it
#pragma unroll
    for (int j = 0; j < 9; ++j) a0 = fma(w[j], v9[j], a0);
    clear();
    couple(cp, 0, 0);  // node q: its elements above, then below
    couple(cm, 4, 4);
    c1 = w[4];
#pragma unroll
    for (int j = 0; j < 9; ++j) a1 = fma(w[j], v9[j], a1);
    clear();
    couple(cp, 4, 0);  // node q + 1 (top corners), plane below it
    a2 = 0.0;
#pragma unroll
    for (int j = 0; j < 9; ++j) a2 = fma(w[j], v9[j], a2);
  };
  auto shift = [&]() {
    a0 = a1;
    a1 = a2;
    c0 = c1;
    xprev = v9[4];
  };
  double preA[4], preB[4];
  double nbA = 0.0, ndA = 0.0, nbB = 0.0, ndB = 0.0;
  load_bd(z0, nbA, ndA);
  load_bd(z0 + 1, nbB, ndB);
  fetch(z0 - 1, preA);
  fetch(z0, preB);
  store(0, z0 - 1, preA);
  store(1, z0, preB);
#pragma unroll
  for (int a = 0; a < 4; ++a) cp[a] = 0.0;
  __syncthreads();
  if (active) {  // planes z0 - 1 and z0: the first two thirds of node z0, the first of z0 + 1
    readn(0);
    add_plane();
    shift();
    readn(1);
    add_plane();
    shift();
  }
  __syncthreads();
  fetch(z0 + 1, preA);
  store(0, z0 + 1, preA);
  fetch(z0 + 2, preA);
  fetch(z0 + 3, preB);
  __syncthreads();
  double contrib = 0.0;
  const bool dxy = active && (((L.mask & 1u) && R.ox + x == 0) || ((L.mask & 2u) && R.ox + x == L.cx - 1) ||
                              ((L.mask & 4u) && R.oy + y == 0) || ((L.mask & 8u) && R.oy + y == L.cy - 1));
  auto plane = [&](int zz, double(&pre)[4], double& b2, double& d2) {
    const int sp = (zz - z0) & 1;  // slot holding plane zz + 1
    const bool work = active && zz < z1;
    if (work) readn(sp);
    if (zz + 2 <= z1) store(sp ^ 1, zz + 2, pre);  // plane zz + 2 replaces plane zz
    fetch(zz + 4, pre);
    const double cb = b2, cd = d2;
    load_bd(zz + 2, b2, d2);
    if (work) {
      add_plane();
      const int64_t gi = R.off + (int64_t)zz * sz + (int64_t)y * sy + x;
      const int gz = R.oz + zz;
      double acc = a0, ctr = c0, xs = xprev;
      if (dxy || ((L.mask & 16u) && gz == 0) || ((L.mask & 32u) && gz == L.cz - 1)) {  // a Dirichlet row
        xs = p.x[gi];
        ctr = sym[coef_index(gi, 0, kSymPts)];
        acc = ctr * xs;
      }
      const bool edge = x == 0 || x == R.ex - 1 || y == 0 || y == R.ey - 1 || zz == 0 || zz == R.ez - 1;
      if (edge && is_shared(L, R, x, y, zz)) write_partial<OP, double>(p, gi, acc, xs, cd);  // finished by k_iface
      else if constexpr (kPreB) contrib += finish_pre<OP, DOT, double, kOwnCentre>(p, gi, acc, 1, xs, ctr, cb, cd);
      else contrib += finish<OP, DOT, double, kOwnCentre>(p, gi, acc, 1, xs, ctr);
      shift();
    }
    __syncthreads();
  };
  // both halves run on every pass, see k_stencil_table
  for (int zz = z0; zz < z1; zz += 2) {
    plane(zz, preA, nbA, ndA);
    plane(zz + 1, preB, nbB, ndB);
  }
  if constexpr (DOT || OP == StencilOp::CgQ) {
    double v = contrib;
    for (int o = 32; o > 0; o >>= 1) v += __shfl_down(v, o, 64);
    __shared__ double sm[NT / 64];
    if ((t & 63) == 0) sm[t >> 6] = v;
    __syncthreads();
    if (t == 0) {
      double s = 0.0;
      for (int i = 0; i < NT / 64; ++i) s += sm[i];
      partials[blockIdx.x] = s;
    }
  }
}

// ----------------------------------------------------------- interface groups
// ng2: the first ng2 groups have two copies each (their copies start at 2 g, no gptr read).
// COPIES: the groups lie on the threads of their first copies in the blocks of k_stencil_fused (a sum is
// then grouped as there).
template <int NDOF, class V, StencilOp OP, bool DOT, bool COPIES>
__global__ __launch_bounds__(kBlock) void k_iface(const int64_t* __restrict__ gptr, const int* __restrict__ gcopy,
                                                  int64_t ng, int64_t ng2, CopyView G, OpP<V> p,
                                                  double* __restrict__ partials) {
  double contrib = 0.0;
  int64_t a0 = 0, e = 0;  // the group's copies
  if constexpr (COPIES) {
    const int first = G.start[blockIdx.x], cnt = G.start[blockIdx.x + 1] - first, t = threadIdx.x;
    if (t < cnt) {
      const int4 ci = G.info[first + t];
      a0 = first + t;
      e = ci.z == t ? a0 + ci.w : a0;
    }
  } else {
    const int64_t g = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    if (g < ng) {
      const bool two = g < ng2;
      a0 = two ? 2 * g : gptr[g];
      e = two ? a0 + 2 : gptr[g + 1];
    }
  }
  if (e > a0) {
    const int m = (int)(e - a0);
    bool block = false;
    if constexpr (NDOF == 3 && (OP == StencilOp::Cheb || OP == StencilOp::ChebFirst)) {
      if (p.dinv9) {  // nodal blocks: the node's three sums first, then the block update
        const int64_t n0 = gcopy[a0];
        V z[3], xs[3], dold[3], out[3], dd[3];
#pragma unroll
        for (int a = 0; a < 3; ++a) {
          V s = (V)0;
          for (int64_t c = a0; c < e; ++c) s += p.out[(int64_t)gcopy[c] * 3 + a];
          z[a] = s;
          xs[a] = p.x[n0 * 3 + a];
          // Cheb: left in p.d by the stencil kernel; ChebFirst: u_(k-1) itself
          dold[a] = OP == StencilOp::Cheb ? p.d[n0 * 3 + a] : xs[a];
        }
        contrib += finish_block3_value<OP, DOT, V>(p, n0, z, xs, dold, out, dd);
        for (int64_t c = a0; c < e; ++c) {
          const int64_t i = (int64_t)gcopy[c] * 3;
#pragma unroll
          for (int a = 0; a < 3; ++a) p.out[i + a] = out[a];
        }
        block = true;
      }
    }
#pragma unroll
    for (int a = 0; a < NDOF; ++a) {
      if (block) break;
      V s = (V)0;
      for (int64_t c = a0; c < e; ++c) s += p.out[(int64_t)gcopy[c] * NDOF + a];
      // the copies of a composite dof hold equal b, x, D~^-1 and previous correction (consistent
      // regional vectors), so the update is computed from the first copy (the lowest region, which
      // owns the dof) and written to every copy
      const int64_t i0 = (int64_t)gcopy[a0] * NDOF + a;
      V out, dd = (V)0;
      const V xs0 = p.x[i0];
      const V dold = OP == StencilOp::Cheb ? p.d[i0] : xs0;  // Cheb: left in p.d by the stencil kernel
      contrib += finish_value<OP, DOT, V>(p, i0, s, m, xs0, (V)0, dold, out, dd);
      for (int64_t c = a0; c < e; ++c) p.out[(int64_t)gcopy[c] * NDOF + a] = out;
    }
  }
  if constexpr (DOT || OP == StencilOp::CgQ) {
    const double s = block_sum(contrib);
    if (threadIdx.x == 0) partials[blockIdx.x] = s;
  }
}

// ------------------------------------------------------------------ dispatch
template <int NPTS, int NDOF, class V, class C, StencilOp OP, bool DOT>
static int64_t run(const Level& L, const StencilArgs& a, hipStream_t st) {
  OpP<V> p{static_cast<const V*>(a.x), static_cast<V*>(a.out), static_cast<const V*>(a.b),
           static_cast<const V*>(a.dinv), static_cast<V*>(a.d), (V)a.c1, (V)a.c2,
           static_cast<const V*>(a.dinv9)};
  const C* coef = a.lowp ? L.coef_lo.as<C>() : L.coef.as<C>();
  const float* centre = L.center_lo.as<float>();
  const LevelView v = L.view();
  constexpr bool kSameType = std::is_same<V, C>::value;
  // the regions' class tables in this arithmetic's type
  const V* table = static_cast<const V*>(a.lowp ? L.class_table_lo.p : L.class_table.p);
  const int* table_ok = a.lowp ? L.class_table_lo_ok.as<int>() : L.class_table_ok.as<int>();
  // region-table split: the served regions' whole-row tiles, then the other regions' element tiles or
  // 2.5D tiles
  const bool elem = NPTS == 27 && NDOF == 1 && std::is_same<V, double>::value && kSameType && !L.elem_tiles.empty();
  const bool split = NPTS == 27 && NDOF == 1 && kSameType && L.use_split && (table || elem) && (!a.lowp || L.split_lo) &&
                     (L.use_tiles || elem || L.other_tiles.empty()) && (OP != StencilOp::CgQ || L.split_dot);
  const bool split3 = NPTS == 27 && NDOF == 3 && L.use_split && table && (!a.lowp || L.split_lo);
  const bool tiled = NPTS == 27 && ((NDOF == 1 && (L.use_tiles || split)) || split3);
  const int ntiles = (int)L.tiles.size();
  const int grid3 = (L.tile_grid > 0 && L.tile_grid < ntiles) ? L.tile_grid : ntiles;
  constexpr bool kSums = DOT || OP == StencilOp::CgQ;
  const bool fused = !tiled && L.fused_stencil(a.lowp);
  int64_t nparts = grid3;  // partial sums written by the tiled launches
  if constexpr (NDOF == 3 && DOT) {
    if (split3) {
      // the sum in a pass of its own: in the step it spilled 30 registers, 446 us on 4.5M nodes, where
      // the step takes 364 and the pass 22
      StencilArgs step = a;
      step.dot_rhs = false;
      run<NPTS, NDOF, V, C, OP, false>(L, step, st);
      return launch_dot(L, static_cast<const double*>(a.b), static_cast<const double*>(a.out), a.partials, st);
    }
  }
  if (a.ev0) RMG_HIP(hipEventRecord(a.ev0, st));
  if constexpr (NPTS == 27 && NDOF == 3 && !DOT) {
    if (split3) {
      nparts = (int64_t)L.table_tiles.size();
      RMG_LAUNCH((k_stencil_table3<V, OP>), dim3(nparts), dim3(kTable3Threads), 0, st, v,
                 L.d_table_tiles.as<Tile3>(), table, p, a.partials);
    }
  }
  if constexpr (NPTS == 27 && NDOF == 1) {
    if (tiled) {
      const C* sym = nullptr;
      if constexpr (kSameType) sym = static_cast<const C*>(a.lowp ? L.coef_lo_sym.p : L.coef_sym.p);
      // tiles by the streaming kernel: n of them at d, partial sums from part on
      auto launch3d = [&](auto nt, int grid, const Tile3* d, int n, double* part) {
        constexpr int NT = decltype(nt)::value;
        if (sym) {
          if constexpr (kSameType) {
            RMG_LAUNCH((k_stencil3d<NT, V, C, OP, DOT, true>), dim3(grid), dim3(NT), 0, st, v, d, n, sym, centre, p,
                       part);
          }
        } else {
          RMG_LAUNCH((k_stencil3d<NT, V, C, OP, DOT, false>), dim3(grid), dim3(NT), 0, st, v, d, n, coef, centre, p,
                     part);
        }
      };
      auto stream = [&](int grid, const Tile3* d, int n, double* part) {
        if constexpr (sizeof(V) == 8) {
          if (L.tile_threads == kTileThreadsF64) launch3d(std::integral_constant<int, kTileThreadsF64>(), grid, d, n, part);
          else launch3d(std::integral_constant<int, kTileThreadsF32>(), grid, d, n, part);
        } else {
          RMG_REQUIRE(L.tile_threads == kTileThreadsF32, RMG_ERR_ARG, "internal: FP32 tiles must be narrow");
          launch3d(std::integral_constant<int, kTileThreadsF32>(), grid, d, n, part);
        }
      };
      if (split) {
        const int64_t nd = (int64_t)L.table_tiles.size(), no = (int64_t)(elem ? L.elem_tiles : L.other_tiles).size();
        RMG_REQUIRE(L.table_served.size() == (size_t)L.nreg, RMG_ERR_ARG, "internal: class tables without their split");
        if constexpr (kSameType) {
          if (nd > 0) {
            auto tables = [&](auto dinv) {
              RMG_LAUNCH((k_stencil_table<V, OP, DOT, decltype(dinv)::value>), dim3(nd), dim3(kTableThreads), 0, st, v,
                         L.d_table_tiles.as<Tile3>(), table, static_cast<const V*>(L.class_dinv_lo.p), p, a.partials);
            };
            if constexpr (sizeof(V) == 4 && (OP == StencilOp::Cheb || OP == StencilOp::ChebFirst)) {
              if (L.use_tiles) tables(std::false_type());
              else tables(std::true_type());
            } else {
              tables(std::false_type());
            }
          }
        }
        if constexpr (kSameType && std::is_same<V, double>::value) {
          if (elem)
            RMG_LAUNCH((k_stencil_elem<OP, DOT>), dim3(no), dim3(kTableThreads), 0, st, v, L.d_elem_tiles.as<Tile3>(),
                       L.elem.as<double>(), L.elem_k, sym, p, a.partials ? a.partials + nd : nullptr);
        }
        if (!elem && no > 0) stream((int)no, L.d_other_tiles.as<Tile3>(), (int)no, a.partials ? a.partials + nd : nullptr);
        nparts = nd + no;
      } else {
        stream(grid3, L.d_tiles.as<Tile3>(), ntiles, a.partials);
      }
    }
  }
  if (!tiled) {
    const C* symc = static_cast<const C*>(a.lowp ? L.coef_lo_sym.p : L.coef_sym.p);
    if (fused) {
      const int nb = (int)L.blocks.size();
      const dim3 g(nb + L.ncopyblk), t(kBlock);
      bool sym = false;
      if constexpr (NPTS == 27) {
        sym = symc != nullptr;
        if (sym)
          RMG_LAUNCH((k_stencil_fused<NPTS, NDOF, V, C, OP, DOT, true>), g, t, 0, st, v, L.copies(), nb, symc, centre, p,
                     a.partials, table, table_ok);
      }
      if (!sym)
        RMG_LAUNCH((k_stencil_fused<NPTS, NDOF, V, C, OP, DOT, false>), g, t, 0, st, v, L.copies(), nb, coef, centre, p,
                   a.partials, (const V*)nullptr, (const int*)nullptr);
      LAUNCH_CHECK();
      if (a.ev1) RMG_HIP(hipEventRecord(a.ev1, st));
      return kSums ? (int64_t)nb + L.ncopyblk : 0;
    }
    auto node = [&](const LevelView& vk, int nblocks, double* part) {
      if constexpr (NPTS == 27) {
        if (symc) {
          RMG_LAUNCH((k_stencil<NPTS, NDOF, V, C, OP, DOT, true>), dim3(nblocks), dim3(kBlock), 0, st, vk,
                             symc, centre, p, part, table, table_ok);
          return;
        }
      }
      RMG_LAUNCH((k_stencil<NPTS, NDOF, V, C, OP, DOT, false>), dim3(nblocks), dim3(kBlock), 0, st, vk, coef,
                         centre, p, part, (const V*)nullptr, (const int*)nullptr);
    };
    if (L.per_region) {
      // unbatched: one launch per region over its slice of the block table (partials keep their slots)
      for (int k = 0; k < L.nreg; ++k) {
        const int b0 = L.region_block[k], b1 = L.region_block[k + 1];
        if (b1 == b0) continue;
        LevelView vk = v;
        vk.blocks = v.blocks + b0;
        vk.nblocks = b1 - b0;
        node(vk, b1 - b0, a.partials ? a.partials + b0 : nullptr);
      }
    } else {
      node(v, (int)L.blocks.size(), a.partials);
    }
  }
  LAUNCH_CHECK();
  if (a.ev1) RMG_HIP(hipEventRecord(a.ev1, st));
  const int64_t nb = tiled ? nparts : (int64_t)L.blocks.size();
  int64_t ngb = 0;
  if (L.ngroups > 0) {
    double* part = a.partials ? a.partials + nb : nullptr;
    // node blocks of a level with copy blocks, whichever of its operations are fused, batched or not: one
    // grouping of the sums
    const bool copies = kSums && !tiled && L.ncopyblk > 0;
    ngb = copies ? L.ncopyblk : cdiv(L.ngroups, kBlock);
    auto iface = [&](auto c) {
      RMG_LAUNCH((k_iface<NDOF, V, OP, DOT, decltype(c)::value>), dim3(ngb), dim3(kBlock), 0, st, L.d_gptr.as<int64_t>(),
                 L.d_gcopy.as<int>(), L.ngroups, L.ngroups2, L.copies(), p, part);
    };
    if constexpr (kSums) {
      if (copies) iface(std::true_type());
      else iface(std::false_type());
    } else {
      iface(std::false_type());
    }
    LAUNCH_CHECK();
  }
  return kSums ? nb + ngb : 0;
}

// FP64: every operation.
template <int NPTS, int NDOF>
static int64_t ops_f64(const Level& L, const StencilArgs& a, hipStream_t st) {
  const bool dot = a.dot_rhs;
  switch (a.op) {
    case StencilOp::Matvec: return run<NPTS, NDOF, double, double, StencilOp::Matvec, false>(L, a, st);
    case StencilOp::Residual: return run<NPTS, NDOF, double, double, StencilOp::Residual, false>(L, a, st);
    case StencilOp::ResidualScaled:
      return run<NPTS, NDOF, double, double, StencilOp::ResidualScaled, false>(L, a, st);
    case StencilOp::Cheb:
      return dot ? run<NPTS, NDOF, double, double, StencilOp::Cheb, true>(L, a, st)
                 : run<NPTS, NDOF, double, double, StencilOp::Cheb, false>(L, a, st);
    case StencilOp::ChebFirst:
      return dot ? run<NPTS, NDOF, double, double, StencilOp::ChebFirst, true>(L, a, st)
                 : run<NPTS, NDOF, double, double, StencilOp::ChebFirst, false>(L, a, st);
    case StencilOp::CgQ: return run<NPTS, NDOF, double, double, StencilOp::CgQ, false>(L, a, st);
  }
  return 0;
}

// FP32 vectors: the V-cycle operations only.
template <int NDOF, class C>
static int64_t ops_f32(const Level& L, const StencilArgs& a, hipStream_t st) {
  RMG_REQUIRE(!a.dot_rhs, RMG_ERR_ARG, "internal: fused dot products need FP64 vectors");
  switch (a.op) {
    case StencilOp::Matvec: return run<27, NDOF, float, C, StencilOp::Matvec, false>(L, a, st);
    case StencilOp::ResidualScaled: return run<27, NDOF, float, C, StencilOp::ResidualScaled, false>(L, a, st);
    case StencilOp::Cheb: return run<27, NDOF, float, C, StencilOp::Cheb, false>(L, a, st);
    case StencilOp::ChebFirst: return run<27, NDOF, float, C, StencilOp::ChebFirst, false>(L, a, st);
    default: fail(RMG_ERR_ARG, "internal: operation not available in FP32");
  }
}

int64_t launch_stencil_op(const Level& L, const StencilArgs& a, hipStream_t st) {
  if (a.lowp) {
    RMG_REQUIRE(L.npts == 27 && L.ct_lo != kCoefF64, RMG_ERR_ARG, "internal: level has no low-precision copy");
    if (L.ndof == 1) return L.ct_lo == kCoefBF16 ? ops_f32<1, uint16_t>(L, a, st) : ops_f32<1, float>(L, a, st);
    return L.ct_lo == kCoefBF16 ? ops_f32<3, uint16_t>(L, a, st) : ops_f32<3, float>(L, a, st);
  }
  if (L.ndof == 3) {
    RMG_REQUIRE(L.npts == 27, RMG_ERR_ARG, "internal: block stencils are 27-point");
    return ops_f64<27, 3>(L, a, st);
  }
  switch (L.npts) {
    case 27: return ops_f64<27, 1>(L, a, st);
    case 9: return ops_f64<9, 1>(L, a, st);
    case 5: return ops_f64<5, 1>(L, a, st);
  }
  fail(RMG_ERR_ARG, "unsupported stencil size");
}

}  // namespace rmg

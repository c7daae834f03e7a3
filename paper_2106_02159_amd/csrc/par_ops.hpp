// par_ops.hpp -- the matrix-free Q1 operators of the parabolic step on a
// uniform box mesh, for one lane per node: neighbour indexing, the
// pre-summed interior stencil and the cell-by-cell element matrix at wall
// nodes (element tables of element.hpp), templated on the value type (FP64
// for the CG, FP32 for the multigrid V-cycle).
#pragma once

#include "par_kernels.hpp"

namespace ns {
namespace pops {

template <int DIM> struct P {
  static constexpr int S = DIM == 2 ? 9 : 27;  // neighbourhood slots
  static constexpr int L = 1 << DIM;           // nodes per cell
  static constexpr int C = S / 2;              // slot of the node itself
};

// (node numbers are below 2^31: unsigned 32-bit division)
__device__ __forceinline__ void decode(const ParGrid &G, int64_t i, int64_t c[3]) {
  const uint32_t n0 = (uint32_t)G.n[0], n1 = (uint32_t)G.n[1];
  const uint32_t t = (uint32_t)i / n0;
  c[0] = (uint32_t)i - t * n0;
  const uint32_t u = t / n1;
  c[1] = t - u * n1;
  c[2] = u;
}

// node at offset (slot s: o_d = (s / 3^d) % 3 - 1) from c, or -1 outside a
// wall-bounded direction
template <int DIM>
__device__ __forceinline__ int64_t nb_index(const ParGrid &G, const int64_t c[3],
                                            int s) {
  int64_t idx = 0, stride = 1;
  int m = 1;
#pragma unroll
  for (int d = 0; d < DIM; ++d) {
    int64_t a = c[d] + (s / m) % 3 - 1;
    m *= 3;
    if (G.per[d]) {
      a = a < 0 ? a + G.n[d] : (a >= G.n[d] ? a - G.n[d] : a);
    } else if (a < 0 || a >= G.n[d]) {
      return -1;
    }
    idx += a * stride;
    stride *= G.n[d];
  }
  return idx;
}

// does the cell in which node c is local node a exist?
template <int DIM>
__device__ __forceinline__ bool cell_exists(const ParGrid &G, const int64_t c[3],
                                            int a) {
  bool ok = true;
#pragma unroll
  for (int d = 0; d < DIM; ++d) {
    const int64_t lo = c[d] - ((a >> d) & 1);
    if (!G.per[d] && (lo < 0 || lo > G.n[d] - 2)) ok = false;
  }
  return ok;
}

// neighbourhood slot of local node b of the cell in which the centre is a
template <int DIM>
__host__ __device__ constexpr int slot_of(int a, int b) {
  int s = 0, m = 1;
  for (int d = 0; d < DIM; ++d) {
    s += (((b >> d) & 1) - ((a >> d) & 1) + 1) * m;
    m *= 3;
  }
  return s;
}

// offsets into the element table (element.hpp, Q1Tables::packed)
template <int DIM> struct TabOff {
  static constexpr int L = 1 << DIM, S = DIM == 2 ? 9 : 27;
  static constexpr int heat = DIM * DIM * L * L;
  static constexpr int phi = heat + L * L;
  static constexpr int dphi = phi + L * L;
  static constexpr int w = dphi + L * L * DIM;
  static constexpr int sst = w + 1;
  static constexpr int sht = sst + S * DIM * DIM;
};

// A node and its neighbours per direction: index contributions at offsets -1,
// 0, 1; a neighbour that does not exist has the node's own.
template <int DIM> struct Near {
  int32_t at[DIM][3];
  Near() = default;
  __device__ __forceinline__ Near(const ParGrid &G, const int64_t c[3]) {
    int32_t stride = 1;
#pragma unroll
    for (int d = 0; d < DIM; ++d) {
      const int32_t n = (int32_t)G.n[d], x = (int32_t)c[d];
      at[d][0] = stride * (x > 0 ? x - 1 : G.per[d] ? n - 1 : x);
      at[d][1] = stride * x;
      at[d][2] = stride * (x < n - 1 ? x + 1 : G.per[d] ? 0 : x);
      stride *= n;
    }
  }
  __device__ __forceinline__ bool lo(int d) const { return at[d][0] != at[d][1]; }
  __device__ __forceinline__ bool hi(int d) const { return at[d][2] != at[d][1]; }
  __device__ __forceinline__ bool interior() const {
    bool in = true;
#pragma unroll
    for (int d = 0; d < DIM; ++d) in = in && lo(d) && hi(d);
    return in;
  }
  // does the cell exist in which the node is local node a?
  __device__ __forceinline__ bool cell(int a) const {
    bool ok = true;
#pragma unroll
    for (int d = 0; d < DIM; ++d) ok = ok && ((a >> d) & 1 ? lo(d) : hi(d));
    return ok;
  }
};

// Tables of the operator with NC components: the stencil and the element
// matrix (entries st[(s NC + k) NC + l], E[((k NC + l) L + a) L + b]).
template <int DIM, int NC, typename T>
__device__ __forceinline__ const T *stencil_of(const T *tab) {
  return tab + (NC > 1 ? TabOff<DIM>::sst : TabOff<DIM>::sht);
}
template <int DIM, int NC, typename T>
__device__ __forceinline__ const T *element_of(const T *tab) {
  return tab + (NC > 1 ? 0 : TabOff<DIM>::heat);
}

// acc_k = (operator row of the node applied to x), without the mass term:
// at interior nodes by the pre-summed 3^dim-point stencil, at wall nodes
// cell by cell with the element matrix (NC = dim: stress, NC = 1: heat).
// get(j, xj) reads the components of x at node j.
// A wall node's lane keeps its whole wave waiting, so its loads are not left
// to a loop over cells and their nodes, one at a time (16 dependent rounds in
// 2D, 64 in 3D): 2D reads the 9 neighbours at once for both forms, 3D a cell's
// 8.  k_cg_apply at 128^3: 267 -> 172 us (stress), 115 -> 60 us (heat); the
// FP32 heat smoother on the levels of 501 x 400: 6.9 -> 4.3 us per iteration.
template <int DIM, int NC, typename T, class TS, class TE, class Get>
__device__ __forceinline__ void op_near(const Near<DIM> &nr, const TS &st, const TE &E,
                                        const Get &get, T (&acc)[NC]) {
  constexpr int L = TabOff<DIM>::L;
#pragma unroll
  for (int k = 0; k < NC; ++k) acc[k] = T(0);
  const bool in = nr.interior();
  if constexpr (DIM == 2) {
    T x[9][NC];
#pragma unroll
    for (int s = 0; s < 9; ++s) get(nr.at[0][s % 3] + nr.at[1][s / 3], x[s]);
    if (in) {
#pragma unroll
      for (int s = 0; s < 9; ++s)
#pragma unroll
        for (int k = 0; k < NC; ++k)
#pragma unroll
          for (int l = 0; l < NC; ++l) acc[k] += st[(s * NC + k) * NC + l] * x[s][l];
    } else {
#pragma unroll
      for (int a = 0; a < L; ++a) {
        if (!nr.cell(a)) continue;
#pragma unroll
        for (int b = 0; b < L; ++b)
#pragma unroll
          for (int k = 0; k < NC; ++k)
#pragma unroll
            for (int l = 0; l < NC; ++l)
              acc[k] += E[((k * NC + l) * L + a) * L + b] * x[slot_of<DIM>(a, b)][l];
      }
    }
  } else {
    if (in) {
      // a plane of 9 neighbours at a time (all 27 gathers in flight at once
      // would cut the occupancy to 2 waves)
#pragma unroll 1
      for (int pl = 0; pl < 3; ++pl) {
        const int32_t z = pl == 0 ? nr.at[2][0] : pl == 1 ? nr.at[2][1] : nr.at[2][2];
        T x[9][NC];
#pragma unroll
        for (int s = 0; s < 9; ++s) get(nr.at[0][s % 3] + nr.at[1][s / 3] + z, x[s]);
#pragma unroll
        for (int s = 0; s < 9; ++s)
#pragma unroll
          for (int k = 0; k < NC; ++k)
#pragma unroll
            for (int l = 0; l < NC; ++l)
              acc[k] += st[((pl * 9 + s) * NC + k) * NC + l] * x[s][l];
      }
    } else {
#pragma unroll 1
      for (int a = 0; a < L; ++a) {
        if (!nr.cell(a)) continue;
        int32_t o[3][2];
#pragma unroll
        for (int d = 0; d < 3; ++d) {
          const bool up = (a >> d) & 1;
          o[d][0] = up ? nr.at[d][0] : nr.at[d][1];
          o[d][1] = up ? nr.at[d][1] : nr.at[d][2];
        }
        T x[8][NC];
#pragma unroll
        for (int b = 0; b < L; ++b) get(o[0][b & 1] + o[1][(b >> 1) & 1] + o[2][b >> 2], x[b]);
#pragma unroll
        for (int b = 0; b < L; ++b)
#pragma unroll
          for (int k = 0; k < NC; ++k)
#pragma unroll
            for (int l = 0; l < NC; ++l)
              acc[k] += E[((k * NC + l) * L + a) * L + b] * x[b][l];
      }
    }
  }
}

template <int DIM, int NC, typename T = double>
__device__ __forceinline__ void op_apply(const ParGrid &G, const T *__restrict__ tab,
                                         const T *__restrict__ x,
                                         const int64_t c[3], T (&acc)[NC]) {
  const int64_t N = G.N;
  const T *__restrict__ st = stencil_of<DIM, NC>(tab);
  const T *__restrict__ E = element_of<DIM, NC>(tab);
  op_near<DIM, NC, T>(Near<DIM>(G, c), st, E, [=](int32_t j, T (&xj)[NC]) {
#pragma unroll
    for (int l = 0; l < NC; ++l) xj[l] = x[l * N + j];
  }, acc);
}

// diagonal entry E^kk_aa summed over the node's cells
template <int DIM, int NC, typename T = double>
__device__ __forceinline__ T op_diag(const ParGrid &G, const T *__restrict__ E,
                                     const int64_t c[3], int k) {
  constexpr int L = P<DIM>::L;
  T d = T(0);
#pragma unroll
  for (int a = 0; a < L; ++a)
    if (cell_exists<DIM>(G, c, a)) d += E[((k * NC + k) * L + a) * L + a];
  return d;
}

}  // namespace pops
}  // namespace ns

// hyp_kernels.hip -- forward-Euler stage of the hyperbolic step on gfx950.
// See hyp_kernels.hpp for the sweep structure and data layout.
#include "hyp_kernels.hpp"

#include "line_sweep.hpp"
#include "row_lists.hpp"

#include <algorithm>
#include <climits>
#include <type_traits>

namespace ns {

namespace {

// aux layout: (a, b) side by side per node, then eta, Phi
template <int DIM> struct Aux {
  static constexpr int AB = 0, ETA = 2, PHI = 3, COUNT = 4;
};
// a and b = a p^(-(gamma-1)/(2 gamma)) of node i
__device__ __forceinline__ double2 aux_ab(const double *__restrict__ aux, int64_t i) {
  return *reinterpret_cast<const double2 *>(aux + 2 * i);
}

// Row width 3^DIM, processed in unrolled chunks of CH slots: the neighbour
// gathers of a chunk are issued together, while the chunk size bounds the
// registers a lane holds (and so the occupancy that hides gather latency).
#ifndef NS_CH_VISC
#define NS_CH_VISC 1
#endif
#ifndef NS_CH_LIM1
#define NS_CH_LIM1 1
#endif
#ifndef NS_CH_LIM2
#define NS_CH_LIM2 1
#endif
#ifndef NS_CH_FIN
#define NS_CH_FIN 1
#endif
// 2D pass-2 search: off-diagonal P_ij kept in LDS instead of registers
#ifndef NS_LIM2_LDS
#define NS_LIM2_LDS 5
#endif
template <int DIM, int CHUNK = 9> struct Cfg {
  static constexpr int NC = DIM + 2;
  static constexpr int W = DIM == 2 ? 9 : 27;
  static constexpr int CH = CHUNK;
  static constexpr int NCH = W / CH;
  static_assert(W % CH == 0, "chunk must divide the row width");
};

// Edge arrays are sliced ELL: rows are grouped in slices of 64 (one
// wavefront) and within a slice stored slot-major, so the 64 lanes of a wave
// reading slot k touch 64 consecutive entries, and all slots of the slice
// share one contiguous block (one page) of every edge array.
template <int DIM>
__device__ __forceinline__ int64_t eidx(int k, int64_t i) {
  constexpr int W = DIM == 2 ? 9 : 27;
  return ((i >> 6) * W + k) * 64 + (i & 63);
}

// Loads of arrays that a sweep reads once per entry (graph coefficients,
// d_ij of the row): with NS_NT they carry the non-temporal hint so
// that they do not push the neighbour rows' node data out of L2.
#ifndef NS_NT
#define NS_NT 2
#endif
template <typename T>
__device__ __forceinline__ T ld_once(global_ptr<const T> p) {
  if constexpr (NS_NT >= 1) return __builtin_nontemporal_load(p);
  else return *p;
}
template <typename T>
__device__ __forceinline__ void st_once(global_ptr<T> p, T v) {
  if constexpr (NS_NT >= 2) __builtin_nontemporal_store(v, p);
  else *p = v;
}
template <typename T>
__device__ __forceinline__ T ld_once(const T *p) {
  if constexpr (NS_NT >= 1) return __builtin_nontemporal_load(p);
  else return *p;
}
template <typename T>
__device__ __forceinline__ void st_once(T *p, T v) {
  if constexpr (NS_NT >= 2) __builtin_nontemporal_store(v, p);
  else *p = v;
}

// Neighbours of row i (in its box mesh); the rows of a workgroup belong to
// one mesh, so the mesh's geometry is a uniform (scalar) load.
// blk is the row block (kBlock rows) of i, uniform over the workgroup.
template <int DIM, typename LT>
__device__ __forceinline__ BoxNbr<DIM> block_nbr(const DevGraphT<LT> &G, uint32_t blk,
                                                 int64_t i) {
  return BoxNbr<DIM>(&G.geo[G.seg ? geo_ld(&G.seg[blk]) : 0], i);
}
// Same for a row that is not the lane's own (work-list entries).
template <int DIM, typename LT>
__device__ __forceinline__ BoxNbr<DIM> row_nbr(const DevGraphT<LT> &G, int64_t i) {
  return BoxNbr<DIM>(&G.geo[G.seg ? G.seg[i / kBlock] : 0], i);
}

__device__ __forceinline__ int64_t row_id() {
  return (int64_t)blockIdx.x * kBlock + threadIdx.x;
}

__device__ __forceinline__ int64_t plain_id() {
  return (int64_t)blockIdx.x * kBlock + threadIdx.x;
}

// Member of a pack that row i belongs to (0 for one mesh).
template <typename LT>
__device__ __forceinline__ int member(const StageArgsT<LT> &A, int64_t i) {
  return A.seg ? A.seg[i / kBlock] : 0;
}

// FP64 value to the storage type: nearest, upwards (graph viscosity stays an
// upper bound) or downwards (a limiter coefficient stays feasible)
template <typename LT> __device__ __forceinline__ LT to_lt(double x) { return (LT)x; }
template <typename LT> __device__ __forceinline__ LT to_lt_up(double x) {
  if constexpr (sizeof(LT) == 4) return __double2float_ru(x);
  else return x;
}
template <typename LT> __device__ __forceinline__ LT to_lt_down(double x) {
  if constexpr (sizeof(LT) == 4) return __double2float_rd(x);
  else return x;
}

// Node vectors in the paired layout of node_layout.hpp: one 16-byte (FP32:
// 8-byte) access per component pair.
template <typename T> struct Pair2;
template <> struct Pair2<double> { using type = double2; };
template <> struct Pair2<float> { using type = float2; };

template <int NC, typename T>
__device__ __forceinline__ void load_state(const T *__restrict__ U,
                                           int64_t N, int64_t i, double *u) {
  using T2 = typename Pair2<T>::type;
#pragma unroll
  for (int p = 0; p < NC / 2; ++p) {
    const T2 v = *reinterpret_cast<const T2 *>(U + 2 * p * N + 2 * i);
    u[2 * p] = v.x;
    u[2 * p + 1] = v.y;
  }
  if constexpr (NC & 1) u[NC - 1] = U[(NC - 1) * N + i];
}

template <int NC, typename T>
__device__ __forceinline__ void store_state(T *__restrict__ U, int64_t N, int64_t i,
                                            const T *u) {
  using T2 = typename Pair2<T>::type;
#pragma unroll
  for (int p = 0; p < NC / 2; ++p) {
    T2 v;
    v.x = u[2 * p];
    v.y = u[2 * p + 1];
    *reinterpret_cast<T2 *>(U + 2 * p * N + 2 * i) = v;
  }
  if constexpr (NC & 1) U[(NC - 1) * N + i] = u[NC - 1];
}

// A line of a node vector (line_sweep.hpp): rows b + off.
template <int NC, typename T>
__device__ __forceinline__ void line_state(const T *__restrict__ U, int64_t N, int64_t b,
                                           uint32_t off, double *u) {
  using T2 = vec2<T>;
#pragma unroll
  for (int p = 0; p < NC / 2; ++p) {
    const T2 v = line_ld(reinterpret_cast<const T2 *>(U + 2 * p * N), b, off);
    u[2 * p] = v.x;
    u[2 * p + 1] = v.y;
  }
  if constexpr (NC & 1) u[NC - 1] = line_ld(U + (NC - 1) * N, b, off);
}

// The value of the neighbour at dx = -1 or +1 from the line's values.
__device__ __forceinline__ double side(int dx, double end, double x) {
  return dx < 0 ? from_left(end, x) : from_right(end, x);
}

// Does the line path handle row i?  (Interior rows; the others are listed.)
template <typename LT>
__device__ __forceinline__ bool line_row(const DevGraphT<LT> &G, int64_t i) {
  return (G.spec[min(i, G.N - 1)] == 0) & (i < G.N);
}

template <typename LT>
__device__ __forceinline__ const BoxGeom *block_geo(const DevGraphT<LT> &G, uint32_t blk) {
  return &G.geo[G.seg ? geo_ld(&G.seg[blk]) : 0];
}

// Entry of slot k of a row of the block that starts at row r0 (a multiple
// of 64), e0 = the lane's entry of slot 0 within the block; and the entry of
// slot k of row jb + tid (jb >= 0 for every active lane's row).
template <int DIM, typename T>
__device__ __forceinline__ global_ptr<T> edge_at(T *a, int64_t r0, int k, uint32_t e0) {
  constexpr int W = DIM == 2 ? 9 : 27;
  return lane_at(a + r0 * W + k * 64, e0);
}
template <int DIM, typename T>
__device__ __forceinline__ global_ptr<T> edge_t(T *a, int64_t jb, int k, uint32_t tid) {
  constexpr int W = DIM == 2 ? 9 : 27;
  // rows counted from the slice boundary below jb
  const uint32_t t = (uint32_t)(jb & 63) + tid;
  const uint32_t e = (t >> 6) * (W * 64) + (t & 63);
  return lane_at(a + (jb >> 6) * (W * 64) + k * 64, e);
}

// Blocks [0, spec_blocks) of a line sweep take the listed rows, the others row
// block blockIdx.x - spec_blocks.  A listed row is shared by the lanes of a
// wave, one per stencil line: on small meshes, where one wave per SIMD hides
// nothing, its 3^d entries one after another took longer than all the rest
// of the launch.
template <int DIM, typename LT>
__host__ __device__ __forceinline__ uint32_t spec_blocks(const DevGraphT<LT> &G) {
  constexpr uint32_t per = (64 / (DIM == 2 ? 3 : 9)) * (kBlock / 64);
  return G.byrow ? 0 : ((uint32_t)G.nsrow + per - 1) / per;
}
// Workgroups of the listed rows, a lane each.
__host__ __device__ __forceinline__ uint32_t spec_slices(int nsrow) {
  return (uint32_t)(nsrow + kBlock - 1) / kBlock;
}
template <int DIM>
struct SpecLane {
  static constexpr int NL = DIM == 2 ? 3 : 9, ROWS = 64 / NL;
  int64_t i;  // row
  int line;   // this lane's line
  int base;   // first lane of the row
  bool ok;    // (lanes without a row repeat another one's, without stores)
  template <typename LT>
  __device__ __forceinline__ explicit SpecLane(const DevGraphT<LT> &G) {
    const int lane = threadIdx.x & 63, grp = lane / NL;
    line = lane - grp * NL;
    base = grp * NL;
    const int t = (int)(blockIdx.x * (kBlock / 64) + threadIdx.x / 64) * ROWS + grp;
    ok = grp < ROWS && t < G.nsrow;
    i = G.srow[min(t, G.nsrow - 1)];
  }
  // Sum and minimum over the row's lines, in line order.
  __device__ __forceinline__ double sum(double x) const {
    double s = 0.0;
#pragma unroll
    for (int l = 0; l < NL; ++l) s += __shfl(x, min(base + l, 63));
    line_keep(s);
    __builtin_amdgcn_sched_barrier(0);  // (one value at a time: registers)
    return s;
  }
  __device__ __forceinline__ double least(double x) const {
    double s = x;
#pragma unroll
    for (int l = 0; l < NL; ++l) s = fmin(s, __shfl(x, min(base + l, 63)));
    return s;
  }
};

__device__ __forceinline__ double block_min(double v) {
  __shared__ double red[kBlock / 64];
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) v = fmin(v, __shfl_xor(v, off));
  const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
  if (lane == 0) red[wid] = v;
  __syncthreads();
  if (threadIdx.x == 0) {
    for (int w = 1; w < kBlock / 64; ++w) v = fmin(v, red[w]);
  }
  return v;
}

// Velocity and pressure of a conserved state; returns the internal energy
// per volume.  The sweeps read whole states and compute them from there.
template <int DIM>
__device__ __forceinline__ double vel_pres(const Gas &g, const double *u, double *v,
                                           double &p) {
#pragma clang fp contract(off)  // the same bits in every kernel
  const double ir = fast_rcp(u[0]);
  double m2 = u[1] * u[1];
#pragma unroll
  for (int k = 1; k < DIM; ++k) m2 = fma(u[1 + k], u[1 + k], m2);
  const double eps = fma(-0.5 * m2, ir, u[DIM + 1]);  // rho e
  p = g.gm1 * eps;
#pragma unroll
  for (int k = 0; k < DIM; ++k) v[k] = u[1 + k] * ir;
  return eps;
}

// ---------------------------------------------------------------------------
template <int DIM>
__device__ __forceinline__ void prim_row(int64_t N, const double *__restrict__ U,
                                         double *__restrict__ aux, const Gas &g,
                                         int64_t i) {
#pragma clang fp contract(off)  // the same bits in every kernel
  if (i >= N) return;
  using X = Aux<DIM>;
  double u[DIM + 2], v[DIM], p;
  load_state<DIM + 2>(U, N, i, u);
  const double r = u[0];
  const double eps = vel_pres<DIM>(g, u, v, p);
  const double a = sqrt(g.gamma * p * (1.0 / r));
  // log p = log(gamma - 1) + log(rho e): one logarithm serves the specific
  // entropy and p^(-(gamma-1)/(2 gamma)) = exp(-ex log p)
  const double le = log(eps);
  const double s = le - g.gamma * log(r);
  double2 ab;
  ab.x = a;
  ab.y = a * exp(-g.ex * (g.lgm1 + le));
  *reinterpret_cast<double2 *>(aux + 2 * i) = ab;
  aux[X::ETA * N + i] = -r * s;
  aux[X::PHI * N + i] = exp(s);
}

template <int DIM>
__global__ __launch_bounds__(kBlock) void k_prim(int64_t N,
                                                 const double *__restrict__ U,
                                                 double *__restrict__ aux,
                                                 Gas g, int *clear) {
  if (clear && blockIdx.x == 0 && threadIdx.x < 4) clear[threadIdx.x] = 0;
  prim_row<DIM>(N, U, aux, g, plain_id());
}

// ---------------------------------------------------------------------------
// Graph viscosity d^L_ij (j > i, stored at (i,j) and (j,i)) and alpha_i.
//
// An interior row and the same row met by the general path (the persistent
// steps) must give the same bits, so the arithmetic of an entry is written
// once, here, with its fused multiply-adds spelled out.  MASK: the
// components of c_ij that can be nonzero (a zero component adds exact
// zeros, so leaving it out changes nothing).
template <int DIM, int MASK>
__device__ __forceinline__ double dot_c(const double *v, const double *c) {
#pragma clang fp contract(off)  // the same bits in every kernel
  double s = 0.0;
  bool first = true;
#pragma unroll
  for (int q = 0; q < DIM; ++q) {
    if (!((MASK >> q) & 1)) continue;
    s = first ? v[q] * c[q] : fma(v[q], c[q], s);
    first = false;
  }
  return s;
}

// f(u) c = (rho v.c, m (v.c) + p c, (v.c)(E + p)); vc = v.c
template <int DIM, int MASK>
__device__ __forceinline__ void flux_c(const double *u, double vc, double p, const double *c,
                                       double *fc) {
#pragma clang fp contract(off)  // the same bits in every kernel
  fc[0] = u[0] * vc;
#pragma unroll
  for (int k = 0; k < DIM; ++k)
    fc[1 + k] = (MASK >> k) & 1 ? fma(u[1 + k], vc, p * c[k]) : u[1 + k] * vc;
  fc[DIM + 1] = vc * (u[DIM + 1] + p);
}

// Entropy variables eta'(U_i) of a row: what its commutator terms need.
template <int DIM>
__device__ __forceinline__ void entropy_vars(const Gas &g, const double *ui, double eps,
                                             double eta, double *etap) {
#pragma clang fp contract(off)  // the same bits in every kernel
  double m2 = ui[1] * ui[1];
#pragma unroll
  for (int k = 1; k < DIM; ++k) m2 = fma(ui[1 + k], ui[1 + k], m2);
  const double s = -eta / ui[0];
  const double ie = 1.0 / eps;
  etap[0] = g.gamma - s - m2 / (2.0 * ui[0] * eps);
#pragma unroll
  for (int k = 0; k < DIM; ++k) etap[1 + k] = ui[1 + k] * ie;
  etap[DIM + 1] = -ui[0] * ie;
}

// Adds entry (i,j) to the indicator's sums N_i, D_i, S_i.
template <int DIM, int MASK>
__device__ __forceinline__ void indicator_term(const double *etap, const double *uj,
                                               const double *vj, double pj, double aj,
                                               double etaj, const double *c, double cn,
                                               double &num, double &den, double &scl) {
#pragma clang fp contract(off)  // the same bits in every kernel
  const double vc = dot_c<DIM, MASK>(vj, c);
  double fc[DIM + 2];
  flux_c<DIM, MASK>(uj, vc, pj, c, fc);
  double t = etaj * vc;
#pragma unroll
  for (int q = 0; q < DIM + 2; ++q) t = fma(-etap[q], fc[q], t);
  num += t;
  den += fabs(t);
  scl = fma(cn * aj, uj[0] + fabs(etaj), scl);
}

// The general path of a row: any boundary, any place.  Row data, and the
// entries of one stencil line (each slot's neighbour gathered on its own;
// absent entries read row i itself, with c = 0).
template <int DIM, int IND>
struct ViscRow {
  static constexpr int NC = DIM + 2;
  double vi[DIM], pi, ai, bi, etap[NC];
  bool wall;
  template <typename LT>
  __device__ __forceinline__ ViscRow(const DevGraphT<LT> &G, const double *__restrict__ U,
                                     const double *__restrict__ aux, const Gas &g, int64_t i) {
    double ui[NC];
    load_state<NC>(U, G.N, i, ui);
    const double2 ab = aux_ab(aux, i);
    ai = ab.x;
    bi = ab.y;
    wall = G.wall[i] != 0;
    const double eps = vel_pres<DIM>(g, ui, vi, pi);
    if constexpr (IND == 0) entropy_vars<DIM>(g, ui, eps, aux[Aux<DIM>::ETA * G.N + i], etap);
  }
};

// Adds the entries of line l to the indicator's sums and stores d_ij for
// j > i.  ANY: the row may be interior (its coefficients are then the
// table's).  SKIP: leave out an entry that none of the wave's rows has.
template <int DIM, int IND, int SEV, bool ANY, bool SKIP, typename LT>
__device__ __forceinline__ void visc_line(const DevGraphT<LT> &G,
                                          const double *__restrict__ U,
                                          const double *__restrict__ aux,
                                          LT *__restrict__ d, const Gas &g,
                                          const BoxNbr<DIM> &jv, int64_t i,
                                          const ViscRow<DIM, IND> &R, int l, bool store,
                                          double &num, double &den, double &scl) {
#pragma clang fp contract(off)  // the same bits in every kernel
  constexpr int NC = DIM + 2, ALL = (1 << DIM) - 1, C = Cfg<DIM>::W / 2;
  const int64_t N = G.N;
  const bool in = ANY && jv.interior();
#pragma unroll 1
  for (int t = 0; t < 3; ++t) {
    const int k = 3 * l + t;
    const int32_t j = jv[k];
    if (SKIP && !__any(j >= 0)) continue;  // (absent entries add zeros)
    const int64_t js = j >= 0 ? j : i;
    double uj[NC];
    load_state<NC>(U, N, js, uj);
    const double2 abj = aux_ab(aux, js);
    const double aj = abj.x, bj = abj.y;
    const double etaj = IND == 0 ? aux[Aux<DIM>::ETA * N + js] : 0.0;
    double c[DIM], vj[DIM], pj;
    jv.grad(k, c);
#pragma unroll
    for (int q = 0; q < DIM; ++q) c[q] = j >= 0 ? c[q] : 0.0;
    vel_pres<DIM>(g, uj, vj, pj);
    const int cls = slot_class<DIM>(k);
    double c2 = c[0] * c[0];
#pragma unroll
    for (int q = 1; q < DIM; ++q) c2 = fma(c[q], c[q], c2);
    double cn = fast_sqrt(c2);
    if (in) cn = jv.g->icn[cls];
    if constexpr (IND == 0)
      indicator_term<DIM, ALL>(R.etap, uj, vj, pj, aj, etaj, c, cn, num, den, scl);
    if (k != C && j > i) {
      double n[DIM];
      const double icn = fast_rcp(cn);
#pragma unroll
      for (int q = 0; q < DIM; ++q) {
        n[q] = c[q] * icn;
        if (in) n[q] = copysign(jv.g->inrm[cls][q], c[q]);
      }
      const double uL = dot_c<DIM, ALL>(R.vi, n), uR = dot_c<DIM, ALL>(vj, n);
      double dij = lambda_max<SEV>(g, uL, R.pi, R.ai, R.bi, uR, pj, aj, bj) * cn;
      if (R.wall) {
        // both ends may be on the wall: c_ji != -c_ij, take both directions
        double ct[DIM];
        grad_transposed<DIM>(k, c, ct);
        double ct2 = ct[0] * ct[0];
#pragma unroll
        for (int q = 1; q < DIM; ++q) ct2 = fma(ct[q], ct[q], ct2);
        const double ctn = fast_sqrt(ct2);
        const double ictn = fast_rcp(ctn);
#pragma unroll
        for (int q = 0; q < DIM; ++q) ct[q] *= ictn;
        dij = fmax(dij, lambda_max<SEV>(g, dot_c<DIM, ALL>(vj, ct), pj, aj, bj,
                                        dot_c<DIM, ALL>(R.vi, ct), R.pi, R.ai, R.bi) * ctn);
      }
      if (store) {
        const LT dst = to_lt_up<LT>(dij);
        st_once(&d[eidx<DIM>(k, i)], dst);
        st_once(&d[eidx<DIM>(tslot<DIM>(k), j)], dst);
      }
    }
  }
}

// alpha_i from its sums (an isolated node -- a padding row of a pack -- has
// den = scl = 0).
template <int IND, typename LT>
__device__ __forceinline__ LT alpha_of(double num, double den, double scl) {
  if constexpr (IND == 0)
    return to_lt<LT>(den + scl > 0.0 ? fabs(num) / fma(1e-2, scl, den) : 0.0);
  return LT(IND == 1 ? 1 : 0);
}

// A listed row, shared by the lanes of its lines.
template <int DIM, int IND, int SEV, typename LT>
__device__ __forceinline__ void visc_spec(const DevGraphT<LT> &G,
                                          const double *__restrict__ U,
                                          const double *__restrict__ aux,
                                          LT *__restrict__ d, LT *__restrict__ alpha,
                                          const Gas &g) {
  const SpecLane<DIM> L(G);
  const ViscRow<DIM, IND> R(G, U, aux, g, L.i);
  double num = 0.0, den = 0.0, scl = 0.0;
  visc_line<DIM, IND, SEV, false, false, LT>(G, U, aux, d, g, row_nbr<DIM>(G, L.i), L.i, R, L.line,
                                      L.ok, num, den, scl);
  num = L.sum(num);
  den = L.sum(den);
  scl = L.sum(scl);
  if (L.ok && L.line == 0) alpha[L.i] = alpha_of<IND, LT>(num, den, scl);
}

// Any row by one lane: sums along the row as the line sweep forms them if it is
// interior, line by line as visc_spec if not.
template <int DIM, int IND, int SEV, bool SKIP, typename LT>
__device__ __forceinline__ void visc_row(const DevGraphT<LT> &G,
                                         const double *__restrict__ U,
                                         const double *__restrict__ aux,
                                         LT *__restrict__ d, LT *__restrict__ alpha,
                                         const Gas &g, BoxNbr<DIM> jv, int64_t i,
                                         bool store = true) {
  const ViscRow<DIM, IND> R(G, U, aux, g, i);
  const bool in = jv.interior();
  double num = 0.0, den = 0.0, scl = 0.0, tn = 0.0, td = 0.0, ts = 0.0;
#pragma unroll 1
  for (int l = 0; l < Cfg<DIM>::W / 3; ++l) {
    visc_line<DIM, IND, SEV, true, SKIP, LT>(G, U, aux, d, g, jv, i, R, l, store, num, den, scl);
    if (!in) {
      tn += num; td += den; ts += scl;
      num = den = scl = 0.0;
    }
  }
  if (store) alpha[i] = in ? alpha_of<IND, LT>(num, den, scl) : alpha_of<IND, LT>(tn, td, ts);
}

// The interior rows of row block blk, line by line (line_sweep.hpp).
template <int DIM, int IND, int SEV, typename LT>
__device__ __forceinline__ void visc_lines(const DevGraphT<LT> &G,
                                           const double *__restrict__ U,
                                           const double *__restrict__ aux,
                                           LT *__restrict__ d, LT *__restrict__ alpha,
                                           const Gas &g, uint32_t blk) {
#pragma clang fp contract(off)  // the same bits in every kernel
  using X = Aux<DIM>;
  constexpr int NC = DIM + 2, W = Cfg<DIM>::W;
  const int64_t N = G.N, r0 = (int64_t)blk * kBlock;
  uint32_t tid = threadIdx.x;
  const uint32_t lane = tid & 63;
  const BoxGeom *geo = block_geo(G, blk);
  const int64_t n0 = geo_ld(&geo->n[0]), n01 = n0 * geo_ld(&geo->n[1]);
  const bool act = line_row(G, r0 + tid);
  const bool edge = ((lane + 1) & 63) < 2;  // lanes 63 and 0
  const Line own = make_line(r0, 0, N, tid);
  double ui[NC], vi[DIM], pi, etap[NC];
  line_state<NC>(U, N, own.b, own.c, ui);
  const vec2<double> abi = line_ld(reinterpret_cast<const vec2<double> *>(aux), own.b, own.c);
  const double etai = IND == 0 ? line_ld(aux + X::ETA * N, own.b, own.c) : 0.0;
  {
    const double eps = vel_pres<DIM>(g, ui, vi, pi);
    if constexpr (IND == 0) entropy_vars<DIM>(g, ui, eps, etai, etap);
  }
  // this lane's entry of slot 0 relative to the block's first edge entry
  const uint32_t e0 = (tid >> 6) * (W * 64) + lane;
  double num = 0.0, den = 0.0, scl = 0.0;
  static_for<0, W / 3>([&](auto line) __attribute__((always_inline)) {
    constexpr int ln = decltype(line)::value;
    constexpr int dy = ln % 3 - 1, dz = DIM == 3 ? ln / 3 - 1 : 0;
    constexpr bool self = dy == 0 && dz == 0;
    // without the indicator only the entries with j > i
    if constexpr (IND != 0 && 3 * ln + 2 <= W / 2) return;
    const int64_t delta = dy * n0 + dz * n01;
    line_fence(tid);
    const Line L = make_line(r0, delta, N, tid);
    double uc[NC], uh[NC], ec, eh = 0.0;
    vec2<double> abc, abh = {0.0, 0.0};
#pragma unroll
    for (int q = 0; q < NC; ++q) uh[q] = 0.0;
    if (self) {
#pragma unroll
      for (int q = 0; q < NC; ++q) uc[q] = ui[q];
      abc = abi;
      ec = etai;
    } else {
      line_state<NC>(U, N, L.b, L.c, uc);
      abc = line_ld(reinterpret_cast<const vec2<double> *>(aux), L.b, L.c);
      ec = IND == 0 ? line_ld(aux + X::ETA * N, L.b, L.c) : 0.0;
    }
    if (edge) {
      line_state<NC>(U, N, L.b, L.h, uh);
      abh = line_ld(reinterpret_cast<const vec2<double> *>(aux), L.b, L.h);
      if (IND == 0) eh = line_ld(aux + X::ETA * N, L.b, L.h);
    }
    static_for<0, 3>([&](auto along) __attribute__((always_inline)) {
      constexpr int dx = decltype(along)::value - 1;
      if constexpr (self && (dx == 0 || (IND != 0 && dx < 0))) return;  // c_ii = 0
      constexpr int k = 3 * ln + dx + 1, cls = slot_class<DIM>(k);
      constexpr int o[3] = {dx, dy, dz};
      double uj[NC], aj, bj, ej;
      if (dx == 0) {
#pragma unroll
        for (int q = 0; q < NC; ++q) uj[q] = uc[q];
        aj = abc.x; bj = abc.y; ej = ec;
      } else {
#pragma unroll
        for (int q = 0; q < NC; ++q) uj[q] = side(dx, uh[q], uc[q]);
        aj = side(dx, abh.x, abc.x);
        bj = side(dx, abh.y, abc.y);
        ej = side(dx, eh, ec);
      }
      double vj[DIM], pj, c[DIM], n[DIM];
      vel_pres<DIM>(g, uj, vj, pj);
#pragma unroll
      for (int q = 0; q < DIM; ++q) {
        c[q] = o[q] < 0 ? -geo_ld(&geo->ic[cls][q]) : geo_ld(&geo->ic[cls][q]);
        n[q] = o[q] < 0 ? -geo_ld(&geo->inrm[cls][q]) : geo_ld(&geo->inrm[cls][q]);
      }
      const double cn = geo_ld(&geo->icn[cls]);
      if constexpr (IND == 0)
        indicator_term<DIM, cls>(etap, uj, vj, pj, aj, ej, c, cn, num, den, scl);
      if constexpr (k > W / 2) {
        const double uL = dot_c<DIM, cls>(vi, n), uR = dot_c<DIM, cls>(vj, n);
        const LT dst =
            to_lt_up<LT>(lambda_max<SEV>(g, uL, pi, abi.x, abi.y, uR, pj, aj, bj) * cn);
        if (act) {
          st_once<LT>(edge_at<DIM>(d, r0, k, e0), dst);
          st_once<LT>(edge_t<DIM>(d, r0 + delta + dx, tslot<DIM>(k), tid), dst);
        }
      }
    });
    line_keep(num, den, scl);
  });
  if (act) alpha[r0 + tid] = alpha_of<IND, LT>(num, den, scl);
}

// FP32 evaluation (mixed-precision mode with FP32 arithmetic, entropy
// indicator, gamma = 7/5): the same quantities as visc_row with the
// velocities, pressures, |c_ij|, the fluxes and commutator terms of the
// indicator and lambda_max in FP32.  d_ij = lambda |c_ij| (1 + 2^-16) rounded
// up stays an upper bound of the FP64 value where lambda_max_f32 certifies
// its error; on the other entries (and for a padding row) lambda_max is
// evaluated in FP64 from the FP64 state, as in visc_row.
template <int DIM>
__device__ __forceinline__ float vel_pres_f(float gm1, const float *u, float *v, float &p) {
  const float ir = __builtin_amdgcn_rcpf(u[0]);
  float m2 = 0.0f;
#pragma unroll
  for (int k = 0; k < DIM; ++k) m2 += u[1 + k] * u[1 + k];
  const float eps = u[DIM + 1] - 0.5f * m2 * ir;
  p = gm1 * eps;
#pragma unroll
  for (int k = 0; k < DIM; ++k) v[k] = u[1 + k] * ir;
  return eps;
}

template <int DIM, typename LT>
__device__ __forceinline__ void visc_row_f32(const DevGraphT<LT> &G,
                                             const double *__restrict__ U,
                                             const double *__restrict__ aux,
                                             LT *__restrict__ d, LT *__restrict__ alpha,
                                             const Gas &g, uint32_t blk, int64_t i) {
  using X = Aux<DIM>;
  using C = Cfg<DIM, NS_CH_VISC>;
  constexpr int NC = C::NC;
  const int64_t N = G.N;
  if (i >= N) return;
  BoxNbr<DIM> jv = block_nbr<DIM>(G, blk, i);
  const float gm1 = (float)g.gm1;
  double ui[NC], vi[DIM], pi;
  load_state<NC>(U, N, i, ui);
  const double eps_i = vel_pres<DIM>(g, ui, vi, pi);  // FP64 (the fallback needs it)
  const double2 abi = aux_ab(aux, i);
  const double ai = abi.x, bi = abi.y;
  const bool wall_i = G.wall[i] != 0;
  // entropy variables of row i, formed in FP64 once per row
  float etap[NC], vif[DIM];
  {
    double m2 = 0.0;
#pragma unroll
    for (int k = 0; k < DIM; ++k) m2 += ui[1 + k] * ui[1 + k];
    const double s = -aux[X::ETA * N + i] / ui[0];
    const double ie = 1.0 / eps_i;
    etap[0] = (float)(g.gamma - s - m2 / (2.0 * ui[0] * eps_i));
#pragma unroll
    for (int k = 0; k < DIM; ++k) {
      etap[1 + k] = (float)(ui[1 + k] * ie);
      vif[k] = (float)vi[k];
    }
    etap[NC - 1] = (float)(-ui[0] * ie);
  }
  const float pif = (float)pi, aif = (float)ai, bif = (float)bi;
  float num = 0.0f, den = 0.0f, scl = 0.0f;
#pragma unroll
  for (int ch = 0; ch < C::NCH; ++ch) {
    jv.fence();
    double c[C::CH][DIM], uj[C::CH][NC], aj[C::CH], bj[C::CH], etaj[C::CH];
    int32_t jc[C::CH];
#pragma unroll
    for (int kk = 0; kk < C::CH; ++kk) {
      const int k = ch * C::CH + kk;
      jc[kk] = jv[k];
      const int64_t js = jc[kk] >= 0 ? jc[kk] : i;
      jv.grad(k, c[kk]);
      const double2 abj = aux_ab(aux, js);
      aj[kk] = abj.x;
      bj[kk] = abj.y;
      load_state<NC>(U, N, js, uj[kk]);
      etaj[kk] = aux[X::ETA * N + js];
    }
#pragma unroll
    for (int kk = 0; kk < C::CH; ++kk) {
      const int k = ch * C::CH + kk;
      const int32_t j = jc[kk];
      if (j < 0) continue;
      float cf[DIM], ujf[NC], vjf[DIM], pjf;
#pragma unroll
      for (int q = 0; q < DIM; ++q) cf[q] = (float)c[kk][q];
#pragma unroll
      for (int q = 0; q < NC; ++q) ujf[q] = (float)uj[kk][q];
      vel_pres_f<DIM>(gm1, ujf, vjf, pjf);
      float c2 = 0.0f, vc = 0.0f;
#pragma unroll
      for (int q = 0; q < DIM; ++q) {
        c2 += cf[q] * cf[q];
        vc += vjf[q] * cf[q];
      }
      const float cn = __builtin_amdgcn_sqrtf(c2);
      {
        // commutator term of the indicator: eta_j (v_j.c) - eta'(U_i).f(U_j) c
        const float etajf = (float)etaj[kk];
        float t = etajf * vc;
        t -= etap[0] * (ujf[0] * vc);
#pragma unroll
        for (int q = 0; q < DIM; ++q) t -= etap[1 + q] * (ujf[1 + q] * vc + pjf * cf[q]);
        t -= etap[NC - 1] * (vc * (ujf[NC - 1] + pjf));
        num += t;
        den += fabsf(t);
        scl += cn * (float)aj[kk] * (ujf[0] + fabsf(etajf));
      }
      if (j > i) {
        const int64_t e = eidx<DIM>(k, i);
        const int kt = tslot<DIM>(k);
        const int64_t et = eidx<DIM>(kt, j);
        const float icn = __builtin_amdgcn_rcpf(cn);
        float uL = 0.0f, uR = 0.0f;
#pragma unroll
        for (int q = 0; q < DIM; ++q) {
          uL += vif[q] * cf[q];
          uR += vjf[q] * cf[q];
        }
        bool ok;
        const float lam = lambda_max_f32(g, uL * icn, pif, aif, bif, uR * icn, pjf,
                                         (float)aj[kk], (float)bj[kk], &ok);
        double dij = (double)lam * (double)cn * kLambdaInflate;
        double vj[DIM], pj;
        if (!ok || wall_i) vel_pres<DIM>(g, uj[kk], vj, pj);
        if (!ok) {  // FP64, as visc_row
          double c2d = 0.0;
#pragma unroll
          for (int q = 0; q < DIM; ++q) c2d += c[kk][q] * c[kk][q];
          const double cnd = fast_sqrt(c2d), icnd = fast_rcp(cnd);
          double uLd = 0.0, uRd = 0.0;
#pragma unroll
          for (int q = 0; q < DIM; ++q) {
            uLd += vi[q] * c[kk][q] * icnd;
            uRd += vj[q] * c[kk][q] * icnd;
          }
          dij = lambda_max<1>(g, uLd, pi, ai, bi, uRd, pj, aj[kk], bj[kk]) * cnd;
        }
        if (wall_i) {
          // both ends may be on the wall: c_ji != -c_ij, take both
          // directions (the transposed one in FP64: walls are a thin set)
          double ct[DIM];
          grad_transposed<DIM>(k, c[kk], ct);
          double ct2 = 0.0;
#pragma unroll
          for (int q = 0; q < DIM; ++q) ct2 += ct[q] * ct[q];
          const double ctn = fast_sqrt(ct2);
          const double ictn = fast_rcp(ctn);
          double uLt = 0.0, uRt = 0.0;
#pragma unroll
          for (int q = 0; q < DIM; ++q) {
            uLt += vj[q] * ct[q] * ictn;
            uRt += vi[q] * ct[q] * ictn;
          }
          dij = fmax(dij, lambda_max<1>(g, uLt, pj, aj[kk], bj[kk], uRt, pi, ai, bi) * ctn);
        }
        const LT dst = to_lt_up<LT>(dij);
        st_once(&d[e], dst);
        st_once(&d[et], dst);
      }
    }
  }
  alpha[i] = to_lt<LT>(den + scl > 0.0f ? fabsf(num) / (den + 1e-2f * scl) : 0.0f);
}

template <int DIM, typename LT>
__global__ __launch_bounds__(kBlock) void k_visc_f32(DevGraphT<LT> G,
                                                     const double *__restrict__ U,
                                                     const double *__restrict__ aux,
                                                     LT *__restrict__ d,
                                                     LT *__restrict__ alpha, Gas g) {
  visc_row_f32<DIM, LT>(G, U, aux, d, alpha, g, blockIdx.x, row_id());
}

template <int DIM, int IND, int SEV, typename LT>
__global__ __launch_bounds__(kBlock) void k_visc(DevGraphT<LT> G,
                                                 const double *__restrict__ U,
                                                 const double *__restrict__ aux,
                                                 LT *__restrict__ d,
                                                 LT *__restrict__ alpha,
                                                 Gas g) {
  const uint32_t ns = spec_blocks<DIM>(G);
  if (blockIdx.x < ns) {
    visc_spec<DIM, IND, SEV, LT>(G, U, aux, d, alpha, g);
  } else {
    visc_lines<DIM, IND, SEV, LT>(G, U, aux, d, alpha, g, blockIdx.x - ns);
  }
}

// A lane's row where every row goes by itself (DevGraphT::byrow; lanes beyond
// the last row repeat it without stores).
template <int DIM>
struct OwnRow {
  int64_t i;
  bool ok;
  BoxNbr<DIM> nb;
  template <typename LT>
  __device__ __forceinline__ explicit OwnRow(const DevGraphT<LT> &G)
      : i(min(row_id(), G.N - 1)), ok(row_id() < G.N), nb(block_nbr<DIM>(G, blockIdx.x, i)) {}
};
template <int DIM, int IND, int SEV, typename LT>
__global__ __launch_bounds__(kBlock) void k_visc_rows(DevGraphT<LT> G,
                                                      const double *__restrict__ U,
                                                      const double *__restrict__ aux,
                                                      LT *__restrict__ d,
                                                      LT *__restrict__ alpha, Gas g) {
  const OwnRow<DIM> r(G);
  visc_row<DIM, IND, SEV, true, LT>(G, U, aux, d, alpha, g, r.nb, r.i, r.ok);
}

// ---------------------------------------------------------------------------
// Time step: per-block min of m_i / (2 sum_{j != i} d_ij) = -m_i / (2 d_ii).
// (every thread of the workgroup calls it: it ends in a workgroup reduction)
template <int DIM, typename LT>
__device__ __forceinline__ void dt_partial_blk(const DevGraphT<LT> &G,
                                               const LT *__restrict__ d,
                                               double *__restrict__ partial, uint32_t blk,
                                               int64_t i) {
  using C = Cfg<DIM>;
  const int64_t N = G.N;
  double r = INFINITY;
  if (i < N) {
    double dsum = 0.0;
    BoxNbr<DIM> jv = block_nbr<DIM>(G, blk, i);
#pragma unroll
    for (int k = 0; k < C::W; ++k) {
      if (k == C::W / 2) continue;  // the diagonal
      const int64_t e = eidx<DIM>(k, i);
      const int32_t j = jv[k];
      const double v = d[e];  // absent entries hold 0
      if (j >= 0 && j != i) dsum += v;
    }
    r = G.mi[i] / (2.0 * dsum);
  }
  r = block_min(r);
  if (threadIdx.x == 0) partial[blk] = r;
}

template <int DIM, typename LT>
__global__ __launch_bounds__(kBlock) void k_dt_partial(DevGraphT<LT> G,
                                                       const LT *__restrict__ d,
                                                       double *__restrict__ partial) {
  dt_partial_blk<DIM, LT>(G, d, partial, blockIdx.x, row_id());
}

// One workgroup per member of a pack: the member's workgroups are
// [mblk[m], mblk[m+1]); min is exact, so tau equals the one-mesh value.
__global__ __launch_bounds__(1024) void k_dt_final_members(const double *__restrict__ partial,
                                                           const int32_t *__restrict__ mblk,
                                                           double cfl,
                                                           double *__restrict__ tau) {
  __shared__ double red[16];
  const int m = blockIdx.x;
  double v = INFINITY;
  for (int64_t b = mblk[m] + threadIdx.x; b < mblk[m + 1]; b += 1024) v = fmin(v, partial[b]);
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) v = fmin(v, __shfl_xor(v, off));
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = v;
  __syncthreads();
  if (threadIdx.x == 0) {
    for (int w = 1; w < 16; ++w) v = fmin(v, red[w]);
    tau[m] = cfl * v;
  }
}

__global__ __launch_bounds__(1024) void k_dt_final(const double *__restrict__ partial,
                                                   int64_t nb, double cfl,
                                                   double *__restrict__ tau) {
  __shared__ double red[16];
  double v = INFINITY;
  for (int64_t b = threadIdx.x; b < nb; b += 1024) v = fmin(v, partial[b]);
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) v = fmin(v, __shfl_xor(v, off));
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = v;
  __syncthreads();
  if (threadIdx.x == 0) {
    for (int w = 1; w < 16; ++w) v = fmin(v, red[w]);
    *tau = cfl * v;
  }
}

// ---------------------------------------------------------------------------
// Low-order update, bounds and high-order flux (stored divided by m_i).
//
// Sums of a row.  sum_j (f(U_j) - f(U_i)) c_ij: the row's own flux enters
// once, against the sum of c_ij over the off-diagonal entries (0 on interior
// rows); only its density component is needed entry by entry, for the bar
// states.
template <int DIM>
struct LoSums {
  static constexpr int NC = DIM + 2;
  double acc[NC], fh[NC], rmin, rmax, phimin, dsum;
};

// Adds entry (i,j): U_j with velocity and pressure, c_ij, d_ij, Phi_j and
// dH_ij.  The arithmetic of interior and other rows, spelled out once.
template <int DIM, int MASK, bool PRED = false>
__device__ __forceinline__ void lo_term(const double *ui, const double *vi, const double *uj,
                                        const double *vj, double pj, const double *c,
                                        double dk, double dH, double phij, LoSums<DIM> &S,
                                        bool there = true) {
#pragma clang fp contract(off)  // the same bits in every kernel
  double fc[DIM + 2];
  flux_c<DIM, MASK>(uj, dot_c<DIM, MASK>(vj, c), pj, c, fc);
  const double vci = dot_c<DIM, MASK>(vi, c);
  // density of the bar state (eq. bar_state) for the local bounds
  double rbar = fma(-fma(-ui[0], vci, fc[0]), fast_rcp(2.0 * dk), 0.5 * (ui[0] + uj[0]));
  if (PRED) rbar = there ? rbar : ui[0];
  S.rmin = fmin(S.rmin, rbar);
  S.rmax = fmax(S.rmax, rbar);
  S.phimin = fmin(S.phimin, phij);
#pragma unroll
  for (int q = 0; q < DIM + 2; ++q) {
    const double du = uj[q] - ui[q];
    S.acc[q] += fma(dk, du, -fc[q]);
    S.fh[q] += fma(dH, du, -fc[q]);
  }
  S.dsum += dk;
}

// U^L, F^H/m_i, bounds and flags of row i from its sums.
template <int DIM, typename LT>
__device__ __forceinline__ void lo_store(const DevGraphT<LT> &G, const StageArgsT<LT> &A,
                                         int64_t i, int mem, double tau, const double *ui,
                                         LT ali, const LoSums<DIM> &S) {
#pragma clang fp contract(off)  // the same bits in every kernel
  constexpr int NC = DIM + 2;
  const int64_t N = G.N;
  const double rmi = G.rmi[i];
  const double tm = tau * rmi;
  double ul[NC];
  LT fs[NC];
#pragma unroll
  for (int q = 0; q < NC; ++q) {
    ul[q] = fma(tm, S.acc[q], ui[q]);
    fs[q] = to_lt<LT>(S.fh[q] * rmi);
  }
  store_state<NC>(A.UL, N, i, ul);
  if constexpr (DIM == 3) {
    // alpha_i beside F^H's fifth component: a neighbour's F^H and alpha come
    // in three 16-byte loads in the limiter sweeps
    LT f6[NC + 1];
#pragma unroll
    for (int q = 0; q < NC; ++q) f6[q] = fs[q];
    f6[NC] = ali;
    store_state<NC + 1>(A.FH, N, i, f6);
  } else {
    store_state<NC>(A.FH, N, i, fs);
  }
  if (A.check_cfl && tau > G.mi[i] / (2.0 * S.dsum)) A.flags[4 * mem] = 1;
  if (A.check_low) {
    double m2 = 0.0;
#pragma unroll
    for (int k = 0; k < DIM; ++k) m2 += ul[1 + k] * ul[1 + k];
    if (!(ul[0] > 0.0) || !(ul[NC - 1] - 0.5 * m2 / ul[0] > 0.0)) A.flags[4 * mem + 3] = 1;
  }
  const double r = G.rrel[i];
  const double bv[3] = {(1.0 - r) * S.rmin, (1.0 + r) * S.rmax, (1.0 - r) * S.phimin};
  store_state<3>(A.bnds, N, i, bv);
}

// first: the lane that empties the limiter work lists of this stage
template <typename LT>
__device__ __forceinline__ void clear_lists(const StageArgsT<LT> &A, bool first) {
  if (first) {
    A.qcnt[0] = 0;
    A.qcnt[1] = 0;
  }
}

// The counters of the stage's limiter: k_lim1's list, 2D the lists' lengths
// (row_lists.hpp), 3D the spread root counters.
template <int DIM, typename LT>
__device__ __forceinline__ void clear_counters(const StageArgsT<LT> &A) {
  clear_lists(A, row_id() == 0);
  if (blockIdx.x == 0 && threadIdx.x < (DIM == 2 ? 64 : 2 * 64)) A.q2[8 * threadIdx.x] = 0;
}

// The general path (see visc_line): adds the entries of line l of row i;
// csum is the sum of c_ij, the diagonal entry's flux goes to F^H directly.
template <int DIM, bool ANY, bool SKIP, typename LT>
__device__ __forceinline__ void lo_line(const DevGraphT<LT> &G, const StageArgsT<LT> &A,
                                        const Gas &g, const BoxNbr<DIM> &jv, int64_t i,
                                        const double *ui, const double *vi, double pi,
                                        double ali, int l, LoSums<DIM> &S, double *csum) {
#pragma clang fp contract(off)  // the same bits in every kernel
  constexpr int NC = DIM + 2, ALL = (1 << DIM) - 1, C = Cfg<DIM>::W / 2;
  const int64_t N = G.N;
  if (SKIP) {  // (absent entries add zeros)
    const bool any = jv[3 * l] >= 0 || jv[3 * l + 1] >= 0 || jv[3 * l + 2] >= 0;
    if (!__any(any)) return;
  }
  double uj[3][NC], phij[3], alj[3], dl[3];
#pragma unroll
  for (int t = 0; t < 3; ++t) {
    const int32_t j = jv[3 * l + t];
    const int64_t js = j >= 0 ? j : i;
    load_state<NC>(A.U, N, js, uj[t]);
    phij[t] = A.aux[Aux<DIM>::PHI * N + js];
    alj[t] = A.alpha[js];
    dl[t] = ld_once(&A.d[eidx<DIM>(3 * l + t, i)]);
  }
#pragma unroll
  for (int t = 0; t < 3; ++t) {
    __builtin_amdgcn_sched_barrier(0);
    const int k = 3 * l + t;
    const bool there = jv[k] >= 0;
    double c[DIM];
    jv.grad(k, c);
    if (k == C) {
      if (!(ANY && jv.interior())) {  // c_ii = 0 there
        double fci[NC];
        flux_c<DIM, ALL>(ui, dot_c<DIM, ALL>(vi, c), pi, c, fci);
#pragma unroll
        for (int q = 0; q < NC; ++q) S.fh[q] -= fci[q];
      }
      continue;
    }
    const double dk = there ? dl[t] : 0.0;
#pragma unroll
    for (int q = 0; q < DIM; ++q) {
      c[q] = there ? c[q] : 0.0;
      csum[q] += c[q];
    }
    double vj[DIM], pj;
    vel_pres<DIM>(g, uj[t], vj, pj);
    lo_term<DIM, ALL, true>(ui, vi, uj[t], vj, pj, c, dk, 0.5 * (ali + alj[t]) * dk, phij[t],
                            S, there);
  }
}

template <int DIM>
__device__ __forceinline__ void lo_clear(LoSums<DIM> &S, double rho, double phi) {
#pragma unroll
  for (int q = 0; q < DIM + 2; ++q) { S.acc[q] = 0.0; S.fh[q] = 0.0; }
  S.rmin = S.rmax = rho;
  S.phimin = phi;
  S.dsum = 0.0;
}

// Adds the row's own flux against the sum of c_ij.
template <int DIM>
__device__ __forceinline__ void lo_own_flux(const double *ui, const double *vi, double pi,
                                            const double *csum, LoSums<DIM> &S) {
#pragma clang fp contract(off)  // the same bits in every kernel
  constexpr int NC = DIM + 2, ALL = (1 << DIM) - 1;
  double fcs[NC];
  flux_c<DIM, ALL>(ui, dot_c<DIM, ALL>(vi, csum), pi, csum, fcs);
#pragma unroll
  for (int q = 0; q < NC; ++q) S.acc[q] += fcs[q];
}

// A listed row, shared by the lanes of its lines.
template <int DIM, typename LT>
__device__ __forceinline__ void lo_spec(const DevGraphT<LT> &G, const StageArgsT<LT> &A,
                                        const Gas &g) {
  constexpr int NC = DIM + 2;
  const SpecLane<DIM> L(G);
  const int64_t i = L.i;
  double ui[NC], vi[DIM], pi, csum[DIM];
  load_state<NC>(A.U, G.N, i, ui);
  vel_pres<DIM>(g, ui, vi, pi);
  const LT al = A.alpha[i];
  LoSums<DIM> S;
  lo_clear(S, ui[0], A.aux[Aux<DIM>::PHI * G.N + i]);
#pragma unroll
  for (int q = 0; q < DIM; ++q) csum[q] = 0.0;
  lo_line<DIM, false, false>(G, A, g, row_nbr<DIM>(G, i), i, ui, vi, pi, (double)al, L.line, S, csum);
#pragma unroll
  for (int q = 0; q < NC; ++q) {
    S.acc[q] = L.sum(S.acc[q]);
    S.fh[q] = L.sum(S.fh[q]);
  }
#pragma unroll
  for (int q = 0; q < DIM; ++q) csum[q] = L.sum(csum[q]);
  S.rmin = L.least(S.rmin);
  S.rmax = -L.least(-S.rmax);
  S.phimin = L.least(S.phimin);
  S.dsum = L.sum(S.dsum);
  lo_own_flux<DIM>(ui, vi, pi, csum, S);
  if (L.ok && L.line == 0) {
    const int mem = member(A, i);
    lo_store<DIM>(G, A, i, mem, A.tau[mem], ui, al, S);
  }
}

// A row by one lane (see visc_row).
template <int DIM, bool SKIP, typename LT>
__device__ __forceinline__ void lo_row(const DevGraphT<LT> &G, const StageArgsT<LT> &A,
                                       const Gas &g, BoxNbr<DIM> jv, int64_t i,
                                       bool store = true) {
  constexpr int NC = DIM + 2;
  double ui[NC], vi[DIM], pi, csum[DIM], tc[DIM];
  load_state<NC>(A.U, G.N, i, ui);
  vel_pres<DIM>(g, ui, vi, pi);
  const LT al = A.alpha[i];
  const int mem = member(A, i);
  const bool in = jv.interior();
  LoSums<DIM> S, T;
  lo_clear(S, ui[0], A.aux[Aux<DIM>::PHI * G.N + i]);
  T = S;
#pragma unroll
  for (int q = 0; q < DIM; ++q) csum[q] = tc[q] = 0.0;
#pragma unroll 1
  for (int l = 0; l < Cfg<DIM>::W / 3; ++l) {
    lo_line<DIM, true, SKIP>(G, A, g, jv, i, ui, vi, pi, (double)al, l, S, csum);
    if (!in) {
#pragma unroll
      for (int q = 0; q < NC; ++q) {
        T.acc[q] += S.acc[q];
        T.fh[q] += S.fh[q];
        S.acc[q] = S.fh[q] = 0.0;
      }
#pragma unroll
      for (int q = 0; q < DIM; ++q) {
        tc[q] += csum[q];
        csum[q] = 0.0;
      }
      T.dsum += S.dsum;
      S.dsum = 0.0;
    }
  }
  if (!in) {
    T.rmin = S.rmin;
    T.rmax = S.rmax;
    T.phimin = S.phimin;
    lo_own_flux<DIM>(ui, vi, pi, tc, T);
    S = T;
  }
  if (store) lo_store<DIM>(G, A, i, mem, A.tau[mem], ui, al, S);
}
template <int DIM, typename LT>
__global__ __launch_bounds__(kBlock) void k_lo_rows(DevGraphT<LT> G, StageArgsT<LT> A, Gas g) {
  clear_counters<DIM>(A);
  const OwnRow<DIM> r(G);
  lo_row<DIM, true>(G, A, g, r.nb, r.i, r.ok);
}

// The interior rows of row block blk, line by line (line_sweep.hpp).
template <int DIM, typename LT>
__device__ __forceinline__ void lo_lines(const DevGraphT<LT> &G, const StageArgsT<LT> &A,
                                         const Gas &g, uint32_t blk) {
#pragma clang fp contract(off)  // the same bits in every kernel
  using X = Aux<DIM>;
  constexpr int NC = DIM + 2, W = Cfg<DIM>::W;
  const int64_t N = G.N, r0 = (int64_t)blk * kBlock;
  uint32_t tid = threadIdx.x;
  const uint32_t lane = tid & 63;
  const BoxGeom *geo = block_geo(G, blk);
  const int64_t n0 = geo_ld(&geo->n[0]), n01 = n0 * geo_ld(&geo->n[1]);
  const bool act = line_row(G, r0 + tid);
  const bool edge = ((lane + 1) & 63) < 2;  // lanes 63 and 0
  const double *__restrict__ U = A.U;
  const double *__restrict__ phi = A.aux + X::PHI * N;
  const LT *__restrict__ alpha = A.alpha;
  const LT *__restrict__ dd = A.d;
  const Line own = make_line(r0, 0, N, tid);
  double ui[NC], vi[DIM], pi;
  line_state<NC>(U, N, own.b, own.c, ui);
  vel_pres<DIM>(g, ui, vi, pi);
  const LT al = line_ld(alpha, own.b, own.c);
  const double ali = al;
  LoSums<DIM> S;
  lo_clear(S, ui[0], line_ld(phi, own.b, own.c));
  const uint32_t e0 = min((tid >> 6), (uint32_t)((N - 1 - r0) >> 6)) * (W * 64) + lane;
  static_for<0, W / 3>([&](auto line) __attribute__((always_inline)) {
    constexpr int ln = decltype(line)::value;
    constexpr int dy = ln % 3 - 1, dz = DIM == 3 ? ln / 3 - 1 : 0;
    constexpr bool self = dy == 0 && dz == 0;
    line_fence(tid);
    const Line L = make_line(r0, dy * n0 + dz * n01, N, tid);
    double uc[NC], uh[NC], ac, ah = 0.0, pc, ph = 0.0, dk[3];
#pragma unroll
    for (int t = 0; t < 3; ++t)
      if (3 * ln + t != W / 2) dk[t] = ld_once<LT>(edge_at<DIM>(dd, r0, 3 * ln + t, e0));
#pragma unroll
    for (int q = 0; q < NC; ++q) uh[q] = 0.0;
    if (self) {
#pragma unroll
      for (int q = 0; q < NC; ++q) uc[q] = ui[q];
      ac = ali;
      pc = line_ld(phi, own.b, own.c);
    } else {
      line_state<NC>(U, N, L.b, L.c, uc);
      ac = line_ld(alpha, L.b, L.c);
      pc = line_ld(phi, L.b, L.c);
    }
    if (edge) {
      line_state<NC>(U, N, L.b, L.h, uh);
      ah = line_ld(alpha, L.b, L.h);
      ph = line_ld(phi, L.b, L.h);
    }
    static_for<0, 3>([&](auto along) __attribute__((always_inline)) {
      constexpr int dx = decltype(along)::value - 1;
      if constexpr (self && dx == 0) return;  // c_ii = 0
      constexpr int k = 3 * ln + dx + 1, cls = slot_class<DIM>(k);
      constexpr int o[3] = {dx, dy, dz};
      double uj[NC], alj, phij;
      if (dx == 0) {
#pragma unroll
        for (int q = 0; q < NC; ++q) uj[q] = uc[q];
        alj = ac; phij = pc;
      } else {
#pragma unroll
        for (int q = 0; q < NC; ++q) uj[q] = side(dx, uh[q], uc[q]);
        alj = side(dx, ah, ac);
        phij = side(dx, ph, pc);
      }
      double vj[DIM], pj, c[DIM];
      vel_pres<DIM>(g, uj, vj, pj);
#pragma unroll
      for (int q = 0; q < DIM; ++q)
        c[q] = o[q] < 0 ? -geo_ld(&geo->ic[cls][q]) : geo_ld(&geo->ic[cls][q]);
      lo_term<DIM, cls>(ui, vi, uj, vj, pj, c, dk[dx + 1], 0.5 * (ali + alj) * dk[dx + 1],
                        phij, S);
      // (one slot at a time: three at once cost a wave per SIMD in 3D)
#pragma unroll
      for (int q = 0; q < NC; ++q) line_keep(S.acc[q], S.fh[q]);
      line_keep(S.rmin, S.rmax, S.phimin, S.dsum);
      if constexpr (DIM == 3) __builtin_amdgcn_sched_barrier(0);
    });
  });
  if (act) {
    const int mem = A.seg ? geo_ld(&A.seg[blk]) : 0;
    lo_store<DIM>(G, A, r0 + tid, mem, A.tau[mem], ui, al, S);
  }
}

template <int DIM, typename LT>
__global__ __launch_bounds__(kBlock) void k_lo(DevGraphT<LT> G, StageArgsT<LT> A, Gas g) {
  clear_counters<DIM>(A);
  const uint32_t ns = spec_blocks<DIM>(G);
  if (blockIdx.x < ns) {
    lo_spec<DIM>(G, A, g);
  } else {
    lo_lines<DIM>(G, A, g, blockIdx.x - ns);
  }
}

// P_ij = tau/(m_i lambda_i) (b_ij F_j - b_ji F_i + (dH - d)(U_j - U_i)) with
// b_ij = -m_ij/m_j, b_ji = -m_ij/m_i (Sec. 3.3); with Fs = F^H/m stored:
// P_ij = tau (|I(i)|-1)/m_i (m_ij (Fs_i - Fs_j) + (dH - d)(U_j - U_i)).
template <int DIM>
struct RowCtx {
  static constexpr int NC = DIM + 2;
  double ui[NC], fi[NC];
  double ali, coef;
};

template <int DIM, typename LT>
__device__ __forceinline__ void load_row(const DevGraphT<LT> &G, const StageArgsT<LT> &A,
                                         int64_t i, double tau, RowCtx<DIM> &R) {
  constexpr int NC = DIM + 2;
  const int64_t N = G.N;
  load_state<NC>(A.U, N, i, R.ui);
  if constexpr (DIM == 3) {
    double f6[NC + 1];
    load_state<NC + 1>(A.FH, N, i, f6);  // F^H / m_i and alpha_i
#pragma unroll
    for (int q = 0; q < NC; ++q) R.fi[q] = f6[q];
    R.ali = f6[NC];
  } else {
    load_state<NC>(A.FH, N, i, R.fi);
    R.ali = A.alpha[i];
  }
  R.coef = tau * G.crm[i];
}

// Neighbour data entering P_ij, gathered unconditionally (absent entries
// read row i itself) so that a chunk's loads are in flight together.
template <int DIM>
struct PIn {
  static constexpr int NC = DIM + 2;
  double u[NC], f[NC], al, d, m;
};

template <int DIM, typename LT>
__device__ __forceinline__ void gather_P(const DevGraphT<LT> &G, const StageArgsT<LT> &A,
                                         int64_t e, int64_t js, double mij, PIn<DIM> &x) {
  constexpr int NC = DIM + 2;
  const int64_t N = G.N;
  load_state<NC>(A.U, N, js, x.u);
  if constexpr (DIM == 3) {
    double f6[NC + 1];
    load_state<NC + 1>(A.FH, N, js, f6);  // F^H / m_j and alpha_j
#pragma unroll
    for (int q = 0; q < NC; ++q) x.f[q] = f6[q];
    x.al = f6[NC];
  } else {
    load_state<NC>(A.FH, N, js, x.f);
    x.al = A.alpha[js];
  }
  x.d = ld_once(&A.d[e]);
  x.m = mij;
}

template <int DIM>
__device__ __forceinline__ void make_P(const RowCtx<DIM> &R, const PIn<DIM> &x,
                                       double *P) {
#pragma clang fp contract(off)  // the same bits in every kernel
  constexpr int NC = DIM + 2;
  const double dH = 0.5 * (R.ali + x.al) * x.d;
#pragma unroll
  for (int q = 0; q < NC; ++q)
    P[q] = R.coef * (x.m * (R.fi[q] - x.f[q]) + (dH - x.d) * (x.u[q] - R.ui[q]));
}

template <int DIM, typename LT>
__device__ __forceinline__ void compute_P(const DevGraphT<LT> &G, const StageArgsT<LT> &A,
                                          const RowCtx<DIM> &R, int64_t e,
                                          int32_t j, double mij, double *P) {
  PIn<DIM> x;
  gather_P<DIM>(G, A, e, j, mij, x);
  make_P<DIM>(R, x, P);
}

template <int DIM, typename LT>
__device__ __forceinline__ void finish(const DevGraphT<LT> &G, const StageArgsT<LT> &A,
                                       int64_t i, const double *u) {
  constexpr int NC = DIM + 2;
  const int64_t N = G.N;
  double w[NC];
  if (A.sa != 0.0) {
    double un[NC];
    load_state<NC>(A.Un, N, i, un);
#pragma unroll
    for (int q = 0; q < NC; ++q) w[q] = fma(A.sa, un[q], A.sb * u[q]);
  } else {
#pragma unroll
    for (int q = 0; q < NC; ++q) w[q] = A.sb * u[q];
  }
  double m2 = 0.0;
#pragma unroll
  for (int k = 0; k < DIM; ++k) m2 += w[1 + k] * w[1 + k];
  const double eps = w[NC - 1] - 0.5 * m2 / w[0];
  if (!(w[0] > 0.0) || !(eps > 0.0)) A.flags[4 * member(A, i) + 1] = 1;
  store_state<NC>(A.out, N, i, w);
}

struct Bounds {
  double rmin, rmax, pmin, pmin5;
};

__device__ __forceinline__ Bounds make_bounds(const double *bv) {
  Bounds b;
  b.rmin = bv[0];
  b.rmax = bv[1];
  b.pmin = bv[2];
  const double p2 = b.pmin * b.pmin;
  b.pmin5 = p2 * p2 * b.pmin;
  return b;
}
template <typename LT>
__device__ __forceinline__ Bounds load_bounds(const StageArgsT<LT> &A, int64_t N,
                                              int64_t i) {
  double bv[3];
  load_state<3>(A.bnds, N, i, bv);  // (rho_min, rho_max) in one load
  return make_bounds(bv);
}

// Limiter line search for every off-diagonal entry of the row.  The cheap
// part (density limit, entropy test at that limit and at 0) runs in the
// row sweep, which stores l = l_rho; entries whose entropy bound cuts inside
// (0, l_rho) are appended to the work list and their root is found by
// k_root.  In a sweep such entries are rare but scattered: solved in place,
// a few lanes would hold their whole wavefront for the length of a root
// search, and the root finder's registers would lower the sweep's occupancy.
template <int DIM, int SEV>
__device__ __forceinline__ int limit_fast(const Gas &g, const double *u,
                                          const double *P, const Bounds &b,
                                          double *l) {
#pragma clang fp contract(off)  // the same bits in every kernel
  double lr = ((P[0] > 0.0 ? b.rmax : b.rmin) - u[0]) / P[0];
  if (!(P[0] > 0.0 || P[0] < 0.0)) lr = 1.0;
  lr = fmin(fmax(lr, 0.0), 1.0);
  *l = lr;
  if (entropy_ok<DIM, SEV>(g, u, P, lr, b.pmin, b.pmin5)) return 0;
  if (!entropy_ok<DIM, SEV>(g, u, P, 0.0, b.pmin, b.pmin5)) { *l = 0.0; return 0; }
  return 1;  // root of psi in (0, lr) still to be found
}

template <int DIM, int SEV, typename LT>
__device__ __forceinline__ void lim1_row(const DevGraphT<LT> &G, const StageArgsT<LT> &A,
                                         const Gas &g, uint32_t blk, int64_t i) {
#pragma clang fp contract(off)  // the same bits in every kernel
  using C = Cfg<DIM, NS_CH_LIM1>;
  constexpr int NC = C::NC;
  const int64_t N = G.N;
  if (i >= N) return;
  BoxNbr<DIM> jv = block_nbr<DIM>(G, blk, i);
  RowCtx<DIM> R;
  load_row<DIM>(G, A, i, A.tau[member(A, i)], R);
  double ul[NC];
  load_state<NC>(A.UL, N, i, ul);
  const Bounds b = load_bounds(A, N, i);
  LT *__restrict__ lt1 = A.lt1;
  uint32_t slow = 0;
#pragma unroll
  for (int ch = 0; ch < C::NCH; ++ch) {
    jv.fence();
    PIn<DIM> x[C::CH];
    int32_t jc[C::CH];
#pragma unroll
    for (int kk = 0; kk < C::CH; ++kk) {
      const int k = ch * C::CH + kk;
      jc[kk] = jv[k];
      if (k == C::W / 2) continue;  // the diagonal has no P
      gather_P<DIM>(G, A, eidx<DIM>(k, i), jc[kk] >= 0 ? jc[kk] : i, jv.mass(k), x[kk]);
    }
#pragma unroll
    for (int kk = 0; kk < C::CH; ++kk) {
      const int k = ch * C::CH + kk;
      if (jc[kk] < 0 || jc[kk] == i) continue;
      double P[NC], l;
      make_P<DIM>(R, x[kk], P);
      if (limit_fast<DIM, SEV>(g, ul, P, b, &l)) slow |= 1u << k;
      st_once(&lt1[eidx<DIM>(k, i)], to_lt_down<LT>(l));
    }
  }
  if (slow) {
    uint32_t t = atomicAdd(&A.qcnt[0], (uint32_t)__builtin_popcount(slow));
    while (slow) {
      const int k = __builtin_ctz(slow);
      slow &= slow - 1;
      A.q[t++] = (uint32_t)eidx<DIM>(k, i);
    }
  }
}

template <int DIM, int SEV, typename LT>
__global__ __launch_bounds__(kBlock) void k_lim1(DevGraphT<LT> G, StageArgsT<LT> A, Gas g) {
  lim1_row<DIM, SEV, LT>(G, A, g, blockIdx.x, row_id());
}

// 3D pass 1: a row's result is (U^L + lambda sum P) less the parts
// lambda (1 - l) P that limiting takes away.  Where those parts are large beside
// the row's own state (a thin gas beside a dense one), their rounding errors
// are too: 5e-14 of the row's state at a density ratio of 1e4, 1e-15 for the
// sum of l P.  share_taken is the size of a part against U^L, the momentum
// against sqrt(2 rho E); rows whose shares add up to more than kMostTaken are
// summed from U^L, every entry l P.  (At 1/2 no row of a Mach-3 shock tube or
// of a field of random jumps of 20 : 1 is, and the errors of the two sums
// agree to 2%.)  A choice between two sums needs no more than FP32.
// k_lim_entries at 192^3: 1.75 -> 1.84 ms per stage.
constexpr float kMostTaken = 0.5f;
template <int DIM>
__device__ __forceinline__ float share_taken(const double *ul, const double *part) {
#pragma clang fp contract(off)  // the same bits in every kernel
  const float rs = __builtin_amdgcn_rsqf((float)ul[0]);
  const float es = __builtin_amdgcn_rsqf((float)ul[DIM + 1]);
  float m = fabsf((float)part[1]);
#pragma unroll
  for (int k = 1; k < DIM; ++k) m = fmaxf(m, fabsf((float)part[1 + k]));
  const float r = fabsf((float)part[0]) * rs * rs, e = fabsf((float)part[DIM + 1]) * es * es;
  return fmaxf(fmaxf(r, e), m * rs * es * 0.70710678f);
}

// MODE 0: convex, pass-1 update + pass-2 line search (2D, the persistent
// steps); 1: convex with one pass, final; 2: l = 1 (unlimited high order),
// final; 3: convex, pass-1 update only (3D, the persistent steps: lim2b_row
// follows, since both at once need more registers than a SIMD lane has).
template <int DIM, int MODE, int SEV, typename LT>
__device__ __forceinline__ void lim2_row(const DevGraphT<LT> &G, const StageArgsT<LT> &A,
                                         const Gas &g, uint32_t blk, int64_t i) {
  // no fused multiply-adds of the compiler's choosing: MODE 0 and 3 must give the
  // bits of the launch path's kernels
#pragma clang fp contract(off)
  using C = Cfg<DIM, NS_CH_LIM2>;
  constexpr int NC = C::NC;
  const int64_t N = G.N;
  if (i >= N) return;
  const LT *__restrict__ lt1 = A.lt1;
  BoxNbr<DIM> colk = block_nbr<DIM>(G, blk, i);
  RowCtx<DIM> R;
  const double tau = A.tau[member(A, i)];
  load_row<DIM>(G, A, i, tau, R);
  const double lam = 1.0 / G.lfac[i];
  double u1[NC];
  load_state<NC>(A.UL, N, i, u1);
  // MODE 3 sums as the launch path does: all of P, less (1 - l) P of the
  // limited pairs (or from U^L, see share_taken); rows that are not interior
  // line by line
  const bool in = MODE == 3 && colk.interior();
  double sub[MODE == 3 ? NC : 1], part[MODE == 3 ? NC : 1], all[MODE == 3 ? NC : 1];
  double ul[MODE == 3 ? NC : 1];
  float taken = 0.0f;
  if constexpr (MODE == 3) {
#pragma unroll
    for (int q = 0; q < NC; ++q) {
      sub[q] = part[q] = all[q] = 0.0;
      ul[q] = u1[q];
    }
  }
  // 2D: the row's P_ij and l_ij stay for the pass-2 search: the P of the
  // first NS_LIM2_LDS off-diagonal slots in the lane's own LDS words (no
  // sharing between lanes, so no barrier), the rest in registers
  constexpr bool CACHE = DIM == 2 && MODE == 0;
  constexpr int NLDS = CACHE ? NS_LIM2_LDS : 0;
  __shared__ double Ps[NLDS > 0 ? NLDS : 1][NC][kBlock];
  const int lane = threadIdx.x;
  double Pc[CACHE ? C::W : 1][NC];
  double lc[CACHE ? C::W : 1];
#pragma unroll
  for (int ch = 0; ch < C::NCH; ++ch) {
    // (the 2D cached form holds fewer registers without the fences)
    if constexpr (!CACHE) colk.fence();
    PIn<DIM> x[C::CH];
    double la[C::CH], lb[C::CH];
    int32_t jc[C::CH];
#pragma unroll
    for (int kk = 0; kk < C::CH; ++kk) {
      const int k = ch * C::CH + kk;
      const int64_t e = eidx<DIM>(k, i);
      jc[kk] = colk[k];
      if (k == C::W / 2) continue;  // the diagonal has no P
      const int64_t js = jc[kk] >= 0 ? jc[kk] : i;
      gather_P<DIM>(G, A, e, js, colk.mass(k), x[kk]);
      if constexpr (MODE != 2) {
        la[kk] = lt1[e];
        lb[kk] = lt1[eidx<DIM>(tslot<DIM>(k), js)];
      }
    }
#pragma unroll
    for (int kk = 0; kk < C::CH; ++kk) {
      const int k = ch * C::CH + kk;
      if (jc[kk] < 0 || jc[kk] == i) continue;
      double P[NC];
      make_P<DIM>(R, x[kk], P);
      const double l = MODE != 2 ? fmin(la[kk], lb[kk]) : 1.0;
      if constexpr (MODE == 3) {
        const double ls = lam * (1.0 - l);
        double off[NC];
#pragma unroll
        for (int q = 0; q < NC; ++q) {
          const double t = lam * P[q];
          if (in) u1[q] += t;
          else part[q] += t;
          off[q] = ls * P[q];
          sub[q] += off[q];
        }
        if (ls != 0.0) taken += share_taken<DIM>(ul, off);
      } else {
#pragma unroll
        for (int q = 0; q < NC; ++q) u1[q] += lam * l * P[q];
      }
      if constexpr (CACHE) {
        const int o = k < C::W / 2 ? k : k - 1;  // off-diagonal ordinal
        if (o < NLDS) {
#pragma unroll
          for (int q = 0; q < NC; ++q) Ps[o < NLDS ? o : 0][q][lane] = P[q];
        } else {
#pragma unroll
          for (int q = 0; q < NC; ++q) Pc[k][q] = P[q];
        }
        lc[k] = l;
      }
    }
    if constexpr (MODE == 3) {
      if ((ch + 1) * C::CH % 3 == 0) {
#pragma unroll
        for (int q = 0; q < NC; ++q) {
          all[q] += part[q];
          part[q] = 0.0;
        }
      }
    }
  }
  if constexpr (MODE == 3) {
#pragma unroll
    for (int q = 0; q < NC; ++q) u1[q] = (in ? u1[q] : u1[q] + all[q]) - sub[q];
    if (taken > kMostTaken) {
#pragma unroll
      for (int q = 0; q < NC; ++q) u1[q] = ul[q];
#pragma unroll 1
      for (int k = 0; k < C::W; ++k) {
        const int32_t j = colk[k];
        if (j < 0 || j == i) continue;
        const int64_t e = eidx<DIM>(k, i);
        PIn<DIM> x;
        double P[NC];
        gather_P<DIM>(G, A, e, j, colk.mass(k), x);
        make_P<DIM>(R, x, P);
        const double ll = lam * fmin((double)lt1[e], (double)lt1[eidx<DIM>(tslot<DIM>(k), j)]);
#pragma unroll
        for (int q = 0; q < NC; ++q) u1[q] += ll * P[q];
      }
    }
    store_state<NC>(A.U1, N, i, u1);
  } else if constexpr (MODE == 1 || MODE == 2) {
    finish<DIM>(G, A, i, u1);
  } else {
    static_assert(CACHE);
    store_state<NC>(A.U1, N, i, u1);
    const Bounds b = load_bounds(A, N, i);
    LT *__restrict__ lt2 = A.lt2;
    uint32_t slow = 0;
    uint32_t nzm = 0;  // slots whose stored product may be nonzero (fin_row)
#pragma unroll
    for (int ch = 0; ch < C::NCH; ++ch) {
      double P[C::CH][NC], l[C::CH];
      int32_t jc[C::CH];
#pragma unroll
      for (int kk = 0; kk < C::CH; ++kk) {
        const int k = ch * C::CH + kk;
        const int o = k < C::W / 2 ? k : k - 1;
        if (k != C::W / 2 && o < NLDS) {
#pragma unroll
          for (int q = 0; q < NC; ++q) P[kk][q] = Ps[o < NLDS ? o : 0][q][lane];
        } else {
#pragma unroll
          for (int q = 0; q < NC; ++q) P[kk][q] = Pc[k][q];
        }
        l[kk] = lc[k];
        jc[kk] = colk[k];
      }
#pragma unroll
      for (int kk = 0; kk < C::CH; ++kk) {
        const int k = ch * C::CH + kk;
        if (jc[kk] < 0 || jc[kk] == i) continue;
        // s1 = 0 (pass 1 took the whole P): the stored product is 0 and a
        // zero direction never needs a root, so the search is skipped
        double l2 = 0.0;
        const double s1 = 1.0 - l[kk];
        if (s1 != 0.0) {
#pragma unroll
          for (int q = 0; q < NC; ++q) P[kk][q] *= s1;
          if (limit_fast<DIM, SEV>(g, u1, P[kk], b, &l2)) slow |= 1u << k;
          else l2 *= s1;
        }
        const LT sv = to_lt_down<LT>(l2);
        st_once(&lt2[eidx<DIM>(k, i)], sv);
        if (sv != LT(0) || ((slow >> k) & 1u)) nzm |= 1u << k;
      }
    }
    A.nzm[i] = nzm;
    if (slow) {
      uint32_t *__restrict__ q2 = A.q2;
      uint32_t t = atomicAdd(&A.qcnt[1], (uint32_t)__builtin_popcount(slow));
      while (slow) {
        const int k = __builtin_ctz(slow);
        slow &= slow - 1;
        q2[t++] = (uint32_t)eidx<DIM>(k, i);
      }
    }
  }
}

template <int DIM, int MODE, int SEV, typename LT>
__global__ __launch_bounds__(kBlock) void k_lim2(DevGraphT<LT> G, StageArgsT<LT> A, Gas g) {
  lim2_row<DIM, MODE, SEV, LT>(G, A, g, blockIdx.x, row_id());
}

// ---------------------------------------------------------------------------
// Two passes (launch path).  First 2D.  Away from shocks the whole of P_ij passes
// both searches of every pair of a row: l_ij = 1, nothing is left for pass 2,
// and the row's result is U^L + lambda_i sum_j P_ij.  So
//   k_lim_first   sweeps along stencil lines: forms every P_ij, tests whether
//                 the row's own search returns 1 (no division: only whether
//                 the step to l = 1 stays inside the bounds), stores that sum
//                 and a mask of the slots where it does not;
//   k_lim_done    finishes the rows whose own and neighbours' masks are clear,
//                 and lists the others (row_lists.hpp);
//   k_lim_rows    runs both limiter passes, roots included, for the marked
//                 rows, 8 lanes (the 8 pairs) to a row;
//   k_fin_rows    adds the pass-2 part of those that have one, 8 lanes to a
//                 row again, or a lane to each of 64 neighbouring rows.
// Marked rows come in long runs, so the waves of k_lim_rows and k_fin_rows take
// equal parts of the list; a wave that worked through its own slice of 64 rows
// had up to 8 rounds of 8 rows, 13 us each, and workgroups with fixed slices all
// over the mesh lined up with fronts.
// Against one sweep that gathered every neighbour slot by slot, kept P for
// pass 2, and listed the entries with a root for two further kernels (FP64,
// limiter and final update of a stage): 2.60 -> 1.33 ms at 4096^2, 0.29 ->
// 0.13 ms at 1001 x 1003, 0.15 -> 0.05 ms at 256^2; there the appends to the
// lists, serial at their counters (15 ns each), and one lane's row of 8
// searches took the time.  k_lim_first is bound by the latency of its line
// loads at 4 waves per SIMD (0.82 ms at 4096^2, 245 B per node: 5.0 TB/s),
// k_lim_done by memory bandwidth (0.27 ms), k_lim_rows by the root finder's
// dependent chain and, where most rows are limited, by its 660 vector
// instructions for 8 rows.  The whole step by the share of rows with jumps
// everywhere (2048^2, one sweep / now): 1% 4.27 / 2.97 ms, 10% 4.45 / 3.21, 50%
// 6.17 / 4.38, 100% 8.38 / 5.40.  The one sweep was ahead only where every row of a
// large mesh is limited and rows are alike along x, so that its lanes never
// diverged: waves along y of 6 nodes, 1500^2, 2.98 / 3.56 ms, of 12 nodes 2.78 /
// 3.05; along x of 6 nodes 5.77 / 5.20.  (A lane per row here, pair by pair, takes
// 3.0 ms for the former's k_lim_rows, not 1.85.)
// Both searches of a pair are evaluated where a row needs them, on operands
// in the order the other row uses, so that both rows obtain the same l_ij
// (as for every kernel here, without fused multiply-adds of the compiler's
// choosing).  KEEP: also store l~, l~' of all entries and U^(1) of all rows
// (the last stage of a step: ns_stats and ns_get_debug read them).

// Does the line search of u + l P return exactly 1?  (x / y >= 1 if and only
// if x >= y for y > 0, also rounded.)
template <int DIM, int SEV>
__device__ __forceinline__ bool limit_is_one(const Gas &g, const double *u, const double *P,
                                             const Bounds &b) {
#pragma clang fp contract(off)
  const bool rho = P[0] > 0.0 ? b.rmax - u[0] >= P[0] : !(P[0] < 0.0) || b.rmin - u[0] <= P[0];
  return entropy_ok<DIM, SEV>(g, u, P, 1.0, b.pmin, b.pmin5) && rho;
}

// F^H / m and alpha of a line (3D: alpha is F^H's sixth component).
template <int DIM, typename LT>
__device__ __forceinline__ void line_flux(const StageArgsT<LT> &A, int64_t N, int64_t b,
                                          uint32_t off, double *f, double &al) {
  constexpr int NC = DIM + 2;
  if constexpr (DIM == 3) {
    double f6[NC + 1];
    line_state<NC + 1>(A.FH, N, b, off, f6);
#pragma unroll
    for (int q = 0; q < NC; ++q) f[q] = f6[q];
    al = f6[NC];
  } else {
    line_state<NC>(A.FH, N, b, off, f);
    al = line_ld(A.alpha, b, off);
  }
}

constexpr int kWide = 512;                  // lanes: 64 rows of 8 pairs

template <int DIM, int SEV, bool KEEP, typename LT>
__device__ __forceinline__ void lim_first_lines(const DevGraphT<LT> &G, const StageArgsT<LT> &A,
                                                const Gas &g, uint32_t blk) {
#pragma clang fp contract(off)
  constexpr int NC = DIM + 2, W = Cfg<DIM>::W;
  const int64_t N = G.N, r0 = (int64_t)blk * kBlock;
  uint32_t tid = threadIdx.x;
  const uint32_t lane = tid & 63;
  const BoxGeom *geo = block_geo(G, blk);
  const int64_t n0 = geo_ld(&geo->n[0]), n01 = n0 * geo_ld(&geo->n[1]);
  const bool act = line_row(G, r0 + tid);
  const bool edge = ((lane + 1) & 63) < 2;  // lanes 63 and 0
  const LT *__restrict__ dd = A.d;
  const Line own = make_line(r0, 0, N, tid);
  RowCtx<DIM> R;
  line_state<NC>(A.U, N, own.b, own.c, R.ui);
  line_flux<DIM>(A, N, own.b, own.c, R.fi, R.ali);
  R.coef = A.tau[A.seg ? geo_ld(&A.seg[blk]) : 0] * line_ld(G.crm, own.b, own.c);
  double ul[NC], u1[NC];
  line_state<NC>(A.UL, N, own.b, own.c, ul);
  Bounds b;
  {
    double bv[3];
    line_state<3>(A.bnds, N, own.b, own.c, bv);
    b = make_bounds(bv);
  }
#pragma unroll
  for (int q = 0; q < NC; ++q) u1[q] = ul[q];
  constexpr double lam = 1.0 / (W - 1);
  uint32_t mask = 0;
  const uint32_t e0 = min((tid >> 6), (uint32_t)((N - 1 - r0) >> 6)) * (W * 64) + lane;
  static_for<0, W / 3>([&](auto line) __attribute__((always_inline)) {
    constexpr int ln = decltype(line)::value;
    constexpr int dy = ln % 3 - 1, dz = DIM == 3 ? ln / 3 - 1 : 0;
    constexpr bool self = dy == 0 && dz == 0;
    line_fence(tid);
    const Line L = make_line(r0, dy * n0 + dz * n01, N, tid);
    double uc[NC], uh[NC], fc[NC], fh[NC], ac, ah = 0.0, dk[3];
#pragma unroll
    for (int t = 0; t < 3; ++t)
      if (3 * ln + t != W / 2) dk[t] = ld_once<LT>(edge_at<DIM>(dd, r0, 3 * ln + t, e0));
#pragma unroll
    for (int q = 0; q < NC; ++q) uh[q] = fh[q] = 0.0;
    if (self) {
#pragma unroll
      for (int q = 0; q < NC; ++q) { uc[q] = R.ui[q]; fc[q] = R.fi[q]; }
      ac = R.ali;
    } else {
      line_state<NC>(A.U, N, L.b, L.c, uc);
      line_flux<DIM>(A, N, L.b, L.c, fc, ac);
    }
    if (edge) {
      line_state<NC>(A.U, N, L.b, L.h, uh);
      line_flux<DIM>(A, N, L.b, L.h, fh, ah);
    }
    static_for<0, 3>([&](auto along) __attribute__((always_inline)) {
      constexpr int dx = decltype(along)::value - 1;
      if constexpr (self && dx == 0) return;  // the diagonal has no P
      constexpr int k = 3 * ln + dx + 1, cls = slot_class<DIM>(k);
      PIn<DIM> x;
#pragma unroll
      for (int q = 0; q < NC; ++q) {
        x.u[q] = dx == 0 ? uc[q] : side(dx, uh[q], uc[q]);
        x.f[q] = dx == 0 ? fc[q] : side(dx, fh[q], fc[q]);
      }
      x.al = dx == 0 ? ac : side(dx, ah, ac);
      x.d = dk[dx + 1];
      x.m = geo_ld(&geo->im[cls]);
      double P[NC];
      make_P<DIM>(R, x, P);
      const bool one = limit_is_one<DIM, SEV>(g, ul, P, b);
      mask |= one ? 0u : 1u << k;
      if constexpr (KEEP)
        if (act) {
          st_once<LT>(edge_at<DIM>(A.lt1, r0, k, e0), LT(1));
          st_once<LT>(edge_at<DIM>(A.lt2, r0, k, e0), LT(0));
        }
#pragma unroll
      for (int q = 0; q < NC; ++q) u1[q] += lam * P[q];
    });
#pragma unroll
    for (int q = 0; q < NC; ++q) line_keep(u1[q]);
    line_keep(mask);
  });
  if (act) {
    store_state<NC>(A.U1, N, r0 + tid, u1);
    A.lim[r0 + tid] = mask;
  }
}

// P_ij of an entry and P_ji as row j forms it: the bracket of P_ji is that
// of P_ij with the sign changed, exactly.
template <int DIM>
__device__ __forceinline__ void make_P_both(const RowCtx<DIM> &R, const PIn<DIM> &x, double cj,
                                            double *P, double *Pj) {
#pragma clang fp contract(off)
  const double dH = 0.5 * (R.ali + x.al) * x.d;
#pragma unroll
  for (int q = 0; q < DIM + 2; ++q) {
    const double B = x.m * (R.fi[q] - x.f[q]) + (dH - x.d) * (x.u[q] - R.ui[q]);
    P[q] = R.coef * B;
    Pj[q] = cj * -B;
  }
}

// A listed row's mask: the own searches, one lane per line; 3D: the sum too
// (2D: k_lim_rows forms it).
template <int DIM, int SEV, bool KEEP, typename LT>
__device__ __forceinline__ void lim_first_spec(const DevGraphT<LT> &G, const StageArgsT<LT> &A,
                                               const Gas &g) {
#pragma clang fp contract(off)
  constexpr int NC = DIM + 2;
  const SpecLane<DIM> L(G);
  const int64_t N = G.N, i = L.i;
  const BoxNbr<DIM> jv = row_nbr<DIM>(G, i);
  RowCtx<DIM> R;
  load_row<DIM>(G, A, i, A.tau[member(A, i)], R);
  double ul[NC], part[NC];
  load_state<NC>(A.UL, N, i, ul);
  const Bounds b = load_bounds(A, N, i);
  const double lam = 1.0 / G.lfac[i];
#pragma unroll
  for (int q = 0; q < NC; ++q) part[q] = 0.0;
  uint32_t mask = 0;
#pragma unroll 1
  for (int t = 0; t < 3; ++t) {
    const int k = 3 * L.line + t;
    const int32_t j = jv[k];
    PIn<DIM> x;
    gather_P<DIM>(G, A, eidx<DIM>(k, i), j >= 0 ? j : i, jv.mass(k), x);
    double P[NC];
    make_P<DIM>(R, x, P);
    if (j >= 0 && j != i) {
      if (!limit_is_one<DIM, SEV>(g, ul, P, b)) mask |= 1u << k;
      if constexpr (DIM == 3) {
#pragma unroll
        for (int q = 0; q < NC; ++q) part[q] += lam * P[q];
        if (KEEP && L.ok) {
          A.lt1[eidx<DIM>(k, i)] = LT(1);
          A.lt2[eidx<DIM>(k, i)] = LT(0);
        }
      }
    }
  }
#pragma unroll
  for (int l = 1; l < SpecLane<DIM>::NL; ++l) mask |= __shfl(mask, min(L.base + l, 63));
  if constexpr (DIM == 3) {
#pragma unroll
    for (int q = 0; q < NC; ++q) part[q] = ul[q] + L.sum(part[q]);
  }
  if (L.ok && L.line == 0) {
    A.lim[i] = mask;
    if constexpr (DIM == 3) store_state<NC>(A.U1, N, i, part);
  }
}

// Every row by itself: the sum in the order of lim_first_lines and, 3D, for a
// row that is not interior of lim_first_spec.
template <int DIM, int SEV, bool KEEP, typename LT>
__global__ __launch_bounds__(kBlock) void k_lim_first_rows(DevGraphT<LT> G, StageArgsT<LT> A,
                                                           Gas g) {
#pragma clang fp contract(off)
  constexpr int NC = DIM + 2, C = Cfg<DIM>::W / 2;
  const OwnRow<DIM> r(G);
  const int64_t N = G.N, i = r.i;
  const BoxNbr<DIM> &jv = r.nb;
  const bool serial = DIM == 2 || jv.interior();
  RowCtx<DIM> R;
  load_row<DIM>(G, A, i, A.tau[member(A, i)], R);
  double ul[NC], u1[NC];
  load_state<NC>(A.UL, N, i, ul);
  const Bounds b = load_bounds(A, N, i);
  const double lam = 1.0 / G.lfac[i];
#pragma unroll
  for (int q = 0; q < NC; ++q) u1[q] = serial ? ul[q] : 0.0;
  uint32_t mask = 0;
#pragma unroll 1
  for (int l = 0; l < Cfg<DIM>::W / 3; ++l) {
    int32_t j[3];
    bool any = false;
    PIn<DIM> x[3];
    double part[NC];
#pragma unroll
    for (int q = 0; q < NC; ++q) part[q] = 0.0;
#pragma unroll
    for (int t = 0; t < 3; ++t) {
      j[t] = 3 * l + t != C ? jv[3 * l + t] : -1;
      any = any || j[t] >= 0;
    }
    if (!__any(any)) continue;
#pragma unroll
    for (int t = 0; t < 3; ++t)
      gather_P<DIM>(G, A, eidx<DIM>(3 * l + t, i), j[t] >= 0 ? j[t] : i, jv.mass(3 * l + t),
                    x[t]);
#pragma unroll
    for (int t = 0; t < 3; ++t) {
      __builtin_amdgcn_sched_barrier(0);
      const int k = 3 * l + t;
      double P[NC];
      make_P<DIM>(R, x[t], P);
      if (j[t] < 0) continue;
      if (!limit_is_one<DIM, SEV>(g, ul, P, b)) mask |= 1u << k;
#pragma unroll
      for (int q = 0; q < NC; ++q) {
        const double t = lam * P[q];
        if (serial) u1[q] += t;
        else part[q] += t;
      }
      if (KEEP && r.ok) {
        A.lt1[eidx<DIM>(k, i)] = LT(1);
        A.lt2[eidx<DIM>(k, i)] = LT(0);
      }
    }
    if (!serial) {
#pragma unroll
      for (int q = 0; q < NC; ++q) u1[q] += part[q];
    }
  }
  if (r.ok) {
    if constexpr (DIM == 3) {
#pragma unroll
      for (int q = 0; q < NC; ++q) u1[q] = serial ? u1[q] : ul[q] + u1[q];
    }
    store_state<NC>(A.U1, N, i, u1);
    A.lim[i] = mask;
  }
}

template <int DIM, int SEV, bool KEEP, typename LT>
__global__ __launch_bounds__(kBlock) void k_lim_first(DevGraphT<LT> G, StageArgsT<LT> A, Gas g) {
  const uint32_t ns = spec_blocks<DIM>(G);
  if (blockIdx.x < ns) lim_first_spec<DIM, SEV, KEEP, LT>(G, A, g);
  else lim_first_lines<DIM, SEV, KEEP, LT>(G, A, g, blockIdx.x - ns);
}

// Both passes of one 2D row by the 8 lanes at `base`: lane o has the o-th
// off-diagonal slot.  Every lane of the wave calls it; lanes with ok = false
// repeat a row without stores.
template <int SEV, bool KEEP, typename LT>
__device__ __forceinline__ void lim_pairs(const DevGraphT<LT> &G, const StageArgsT<LT> &A,
                                          const Gas &g, int64_t i, int o, int base, bool ok,
                                          uint32_t *roots, double *nb_words) {
#pragma clang fp contract(off)
  constexpr int NC = 4;
  const int64_t N = G.N;
  const BoxNbr<2> nb = row_nbr<2>(G, i);
  const int k = o < 4 ? o : o + 1;
  const int32_t j = nb[k];
  const bool there = j >= 0;
  const int64_t js = there ? j : i, e = eidx<2>(k, i);
  const double tau = A.tau[member(A, i)];
  RowCtx<2> R;
  PIn<2> x;
  load_row<2>(G, A, i, tau, R);
  gather_P<2>(G, A, e, js, nb.mass(k), x);
  double ul[NC], uj[NC], P[NC], Pj[NC];
  load_state<NC>(A.UL, N, i, ul);
  load_state<NC>(A.UL, N, js, uj);
  const Bounds b = load_bounds(A, N, i), bj = load_bounds(A, N, js);
  make_P_both<2>(R, x, tau * G.crm[js], P, Pj);
  const double lam = 1.0 / G.lfac[i];
  // Pass 1: the pair's two searches; pass 2: the search on (1 - l) P from the
  // updated row.  `pend`: a bit for each search that needs the root (0 own,
  // 1 neighbour's, 2 pass 2).  The root finder is one body and runs for every
  // lane's next one at once: few pairs have two.  The neighbour's operands
  // wait in the lane's LDS words (in registers they were spilled inside the
  // root finder's loops).
  double l = 1.0, s1 = 1.0, u1[NC], own = 1.0, rj = 1.0, l2 = 0.0;
  uint32_t pend = 0;
  if (there && limit_fast<2, SEV>(g, uj, Pj, bj, &rj)) {
    pend = 2;
#pragma unroll
    for (int q = 0; q < NC; ++q) {
      nb_words[q * kWide] = uj[q];
      nb_words[(NC + q) * kWide] = Pj[q];
    }
    nb_words[2 * NC * kWide] = bj.pmin;
  }
  bool slow1 = false, slow2 = false;
#pragma unroll
  for (int q = 0; q < NC; ++q) u1[q] = ul[q];
#pragma unroll 1
  for (int pass = 0; pass < 2; ++pass) {
    double r0 = pass ? 0.0 : 1.0;
    if (there && s1 != 0.0 && limit_fast<2, SEV>(g, u1, P, b, &r0)) pend |= 1;
    if (pass) slow2 = pend & 1;
    else slow1 = pend & 1;
#pragma unroll 1
    while (__any(pend)) {
      const bool nbr = pend == 2;
      double us[NC], Ps[NC], pm = b.pmin;
#pragma unroll
      for (int q = 0; q < NC; ++q) {
        us[q] = u1[q];
        Ps[q] = P[q];
      }
      if (nbr) {
#pragma unroll
        for (int q = 0; q < NC; ++q) {
          us[q] = nb_words[q * kWide];
          Ps[q] = nb_words[(NC + q) * kWide];
        }
        pm = nb_words[2 * NC * kWide];
      }
      if (pend) {
        const double p2 = pm * pm;
        // (the bracket as the sweeps store it)
        const double lr = (double)to_lt_down<LT>(nbr ? rj : r0);
        const double r = entropy_root_fast<2, SEV>(g, us, Ps, lr, pm, p2 * p2 * pm);
        if (nbr) rj = r;
        else r0 = r;
        pend &= pend - 1;
      }
    }
    if (pass == 0) {
      own = (double)to_lt_down<LT>(r0);
      l = fmin(own, (double)to_lt_down<LT>(rj));
      s1 = 1.0 - l;  // (0: the stored product is 0)
#pragma unroll
      for (int q = 0; q < NC; ++q) {
        const double t = there ? lam * l * P[q] : 0.0;
#pragma unroll
        for (int p = 0; p < 8; ++p) u1[q] += __shfl(t, base + p);  // in slot order
        P[q] *= s1;
      }
    } else {
      l2 = r0 * s1;
    }
  }
  const LT sv = to_lt_down<LT>(l2);
  if (ok && there) {
    if constexpr (KEEP) A.lt1[e] = (LT)own;
    if (KEEP || sv != LT(0)) A.lt2[e] = sv;
  }
  const uint64_t nzw = __ballot(ok && there && sv != LT(0));
  const uint32_t m8 = (uint32_t)(nzw >> base) & 0xffu, nz = (m8 & 15u) | (m8 >> 4) << 5;
  if constexpr (KEEP) {  // entries that needed the root finder
    const int n1 = __builtin_popcountll(__ballot(ok && slow1));
    const int n2 = __builtin_popcountll(__ballot(ok && slow2));
    if ((threadIdx.x & 63) == 0 && (n1 | n2)) {
      atomicAdd(&roots[0], (uint32_t)n1);
      atomicAdd(&roots[1], (uint32_t)n2);
    }
  }
  if (ok && o == 0) {
    A.nzm[i] = nz;
    if (KEEP || nz) store_state<NC>(A.U1, N, i, u1);
    if (!nz) finish<2>(G, A, i, u1);
  }
}

// Inclusive sum over the lanes of a wave.
__device__ __forceinline__ uint32_t wave_scan(uint32_t c, uint32_t lane) {
#pragma unroll
  for (int d = 1; d < 64; d <<= 1) {
    const uint32_t o = __shfl_up(c, d);
    if ((int)lane >= d) c += o;
  }
  return c;
}

// Workgroups of k_lim_rows beside those of the listed rows: two per CU (what
// fits), or one to 64 rows of a small mesh.
__host__ __device__ __forceinline__ uint32_t lim_groups(int64_t N) {
  const int64_t sl = (N + 63) / 64;
  return (uint32_t)(sl < 512 ? sl : 512);
}
__host__ __device__ __forceinline__ uint32_t row_blocks(int64_t N) {
  return (uint32_t)((N + kListRows - 1) / kListRows);
}
template <typename LT>
__host__ __device__ __forceinline__ uint32_t spec_groups(const DevGraphT<LT> &G) {
  return G.byrow ? 0 : (uint32_t)(G.nsrow + 63) / 64;
}
// A.q2: the lists' lengths, then (KEEP) the root counts of k_lim_rows'
// workgroups.
constexpr uint32_t kRootWords = kMaxLists * kListStep;

// Appends the marked lanes' rows of a workgroup to its list in A.q (every thread
// calls it).
template <typename LT>
__device__ __forceinline__ void list_rows(const DevGraphT<LT> &G, const StageArgsT<LT> &A,
                                          int64_t i, bool marked) {
  __shared__ uint32_t cnt[kBlock / 64], at;
  const uint32_t tid = threadIdx.x;
  const uint64_t w = __ballot(marked);
  if ((tid & 63) == 0) cnt[tid >> 6] = (uint32_t)__builtin_popcountll(w);
  __syncthreads();
  uint32_t total = 0, before = 0;
#pragma unroll
  for (uint32_t v = 0; v < kBlock / 64; ++v) {
    before += v < (tid >> 6) ? cnt[v] : 0;
    total += cnt[v];
  }
  if (total == 0) return;
  const RowLists rl(row_blocks(G.N));
  const uint32_t list = rl.list_of(blockIdx.x);
  if (tid == 0) at = atomicAdd(&A.q2[kListStep * list], total);
  __syncthreads();
  if (marked)
    A.q[(int64_t)list * rl.room + at + before +
        __builtin_amdgcn_mbcnt_hi((uint32_t)(w >> 32),
                                  __builtin_amdgcn_mbcnt_lo((uint32_t)w, 0))] = (uint32_t)i;
}

// Finishes the interior rows without a limited pair and lists the others.
template <typename LT>
__global__ __launch_bounds__(kBlock) void k_lim_done(DevGraphT<LT> G, StageArgsT<LT> A) {
  const int64_t N = G.N, r0 = (int64_t)blockIdx.x * kBlock;
  const uint32_t tid = threadIdx.x;
  const int lane = tid & 63;
  const int64_t n0 = geo_ld(&block_geo(G, blockIdx.x)->n[0]);
  const bool act = line_row(G, r0 + tid);
  const bool edge = ((lane + 1) & 63) < 2;
  uint32_t mc[3], mh[3] = {0, 0, 0};
#pragma unroll
  for (int ln = 0; ln < 3; ++ln) {
    const Line L = make_line(r0, (ln - 1) * n0, N, tid);
    mc[ln] = line_ld(A.lim, L.b, L.c);
    if (edge) mh[ln] = line_ld(A.lim, L.b, L.h);
  }
  double u1[4];
  const Line own = make_line(r0, 0, N, tid);
  line_state<4>(A.U1, N, own.b, own.c, u1);
  uint32_t lim = mc[1];
#pragma unroll
  for (int ln = 0; ln < 3; ++ln) {
    // slot k of this row is slot 8 - k of the neighbour's
    lim |= (from_left(mh[ln], mc[ln]) >> (8 - 3 * ln)) & 1u;
    if (ln != 1) lim |= (mc[ln] >> (7 - 3 * ln)) & 1u;
    lim |= (from_right(mh[ln], mc[ln]) >> (6 - 3 * ln)) & 1u;
  }
  if (act) {
    A.nzm[r0 + tid] = 0;
    if (lim == 0) finish<2>(G, A, r0 + tid, u1);
  }
  list_rows(G, A, r0 + tid, act && lim != 0);
}

// Every row by itself.
template <typename LT>
__global__ __launch_bounds__(kBlock) void k_lim_done_rows(DevGraphT<LT> G, StageArgsT<LT> A) {
  const OwnRow<2> r(G);
  uint32_t lim = A.lim[r.i];
#pragma unroll
  for (int k = 0; k < 9; ++k) {
    const int32_t j = r.nb[k];
    if (k != 4) lim |= j >= 0 ? (A.lim[j >= 0 ? j : r.i] >> (8 - k)) & 1u : 0u;
  }
  if (r.ok) {
    A.nzm[r.i] = 0;
    if (lim == 0) {
      double u1[4];
      load_state<4>(A.U1, G.N, r.i, u1);
      finish<2>(G, A, r.i, u1);
    }
  }
  list_rows(G, A, r.i, r.ok && lim != 0);
}

struct NoRows {};
// f(row, ok) for the rows of this wave, 8 at a time (a lane's row is lane / 8's;
// lanes with ok = false have another one's): of G.srow in the first `ns`
// workgroups, of the lists in the others.  all(row, ok): offered 64 rows, a lane
// each, where a workgroup has 512 rows to a round; false: not taken.
template <typename LT, class F, class M>
__device__ __forceinline__ void wave_rows(const DevGraphT<LT> &G, const StageArgsT<LT> &A,
                                          uint32_t ns, F &&f, M &&all) {
  const uint32_t lane = threadIdx.x & 63;
  const uint32_t wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const bool front = blockIdx.x < ns;
  uint32_t lists = 1, room = 0, each = 64, step = 1, len = (uint32_t)G.nsrow, longest = len;
  const uint32_t *q = (const uint32_t *)G.srow;
  if (!front) {
    const RowLists rl(row_blocks(G.N));
    const uint32_t groups = lim_groups(G.N);
    lists = rl.lists;
    room = rl.room;
    q = A.q;
    step = groups;
    len = lane < lists ? A.q2[kListStep * lane] : 0;
    longest = len;
#pragma unroll
    for (int d = 32; d > 0; d >>= 1) longest = max(longest, (uint32_t)__shfl_xor((int)longest, d));
    longest = __builtin_amdgcn_readfirstlane(longest);
    each = part_rows(longest, lists, groups);
  }
  if constexpr (!std::is_same_v<M, NoRows>) {
    if (!front && longest * lists / 512 >= step) {
      for (uint32_t p = blockIdx.x - ns;; p += step) {
        const uint32_t l = p & (lists - 1), at = p / lists * 512 + 64 * wave;
        if (p / lists * 512 >= longest) return;
        const uint32_t n = __builtin_amdgcn_readlane(len, l);
        if (at >= n) continue;
        const uint32_t *__restrict__ r = q + (int64_t)l * room;
        if (all(r[min(at + lane, n - 1)], at + lane < n)) continue;
  #pragma unroll 1
        for (uint32_t t0 = at; t0 < min(at + 64, n); t0 += 8) {
          const uint32_t t = t0 + (lane >> 3);
          f(r[min(t, n - 1)], t < n);
        }
      }
    }
  }
  if (8 * wave >= each) return;
  for (uint32_t p = front ? blockIdx.x : blockIdx.x - ns;; p += step) {
    const uint32_t l = p & (lists - 1), at = p / lists * each;
    if (at >= longest) return;
    const uint32_t n = __builtin_amdgcn_readlane(len, l), t0 = at + 8 * wave;
    if (t0 < n) {
      const uint32_t t = t0 + (lane >> 3);
      f(q[(int64_t)l * room + min(t, n - 1)], t < n);
    }
    if (front) return;
  }
}

// The listed rows (front workgroups; none where every row goes by itself), and
// the marked rows, 8 to a wave.
template <int SEV, bool KEEP, typename LT>
__global__ __launch_bounds__(kWide) __attribute__((amdgpu_waves_per_eu(4, 4))) void k_lim_rows(
    DevGraphT<LT> G, StageArgsT<LT> A, Gas g) {
  __shared__ double nb_words[9][kWide];
  __shared__ uint32_t roots[2];
  const uint32_t ns = spec_groups(G), tid = threadIdx.x;
  const uint32_t lane = tid & 63;
  if constexpr (KEEP) {
    if (tid < 2) roots[tid] = 0;
    __syncthreads();
  }
  wave_rows(G, A, ns, [&](uint32_t row, bool ok) __attribute__((always_inline)) {
    lim_pairs<SEV, KEEP, LT>(G, A, g, row, lane & 7, lane & ~7u, ok, roots, &nb_words[0][tid]);
  }, NoRows());
  if constexpr (KEEP) {
    __syncthreads();
    if (tid < 2) A.q2[kRootWords + 2 * blockIdx.x + tid] = roots[tid];
  }
}

// U = U^(1) + lambda_i sum l' (1 - l) P of a limited row with a pass-2 part,
// by the 8 lanes at `base` (see lim_pairs), in slot order.  A product that
// its row did not store is 0 (its mask bit is clear).
template <typename LT>
__device__ __forceinline__ void fin_pairs(const DevGraphT<LT> &G, const StageArgsT<LT> &A,
                                          int64_t i, int o, int base, bool ok) {
#pragma clang fp contract(off)
  constexpr int NC = 4;
  const int64_t N = G.N;
  const int k = o < 4 ? o : o + 1;
  const uint32_t nz = A.nzm[i];
  ok = ok && nz != 0;
  double t[NC];
#pragma unroll
  for (int q = 0; q < NC; ++q) t[q] = 0.0;
  if (ok && ((nz >> k) & 1u)) {
    const BoxNbr<2> jv = row_nbr<2>(G, i);
    const int32_t j = jv[k];
    const int64_t e = eidx<2>(k, i), et = eidx<2>(tslot<2>(k), j);
    const double la = A.lt2[e], lb = A.lt2[et];
    RowCtx<2> R;
    load_row<2>(G, A, i, A.tau[member(A, i)], R);
    PIn<2> x;
    gather_P<2>(G, A, e, j, jv.mass(k), x);
    const double w = (A.nzm[j] >> tslot<2>(k)) & 1u ? 1.0 / G.lfac[i] * fmin(la, lb) : 0.0;
    double P[NC];
    make_P<2>(R, x, P);
#pragma unroll
    for (int q = 0; q < NC; ++q) t[q] = w * P[q];
  }
  double u2[NC];
  load_state<NC>(A.U1, N, i, u2);
#pragma unroll
  for (int q = 0; q < NC; ++q)
#pragma unroll
    for (int p = 0; p < 8; ++p) u2[q] += __shfl(t[q], base + p);
  if (ok && o == 0) finish<2>(G, A, i, u2);
}

// The same for 64 rows, a lane each, slot by slot: where the rows follow one
// another and a slot that any of them has is one that at least kFilled of them
// have, lanes without work cost less than eight lanes' loads of a row's own
// data.  All rows limited, 1500 x 1500, k_fin_rows per stage: waves along y (6
// nodes) 0.39 -> 0.13 ms, 1% noise on the Mach-3 tube (1000 x 1000) 0.16 -> 0.15;
// with 24 or 32 in place of 16 the former takes 0.16 and 0.17, and without the
// rule jumps everywhere take 0.29, not 0.18.  Returns false if the rows are not so.
constexpr uint32_t kFilled = 16;
template <typename LT>
__device__ __forceinline__ bool fin_dense(const DevGraphT<LT> &G, const StageArgsT<LT> &A,
                                          int64_t i, bool ok) {
#pragma clang fp contract(off)
  constexpr int NC = 4;
  const uint32_t nz = ok ? A.nzm[i] : 0;
  if (!__any(nz)) return true;
  uint32_t bits = (uint32_t)__builtin_popcount(nz), slots = nz;
#pragma unroll
  for (int d = 32; d > 0; d >>= 1) {
    bits += __shfl_xor(bits, d);
    slots |= __shfl_xor(slots, d);
  }
  const uint64_t next = __ballot(__shfl_down((int)i, 1) == (int)i + 1);
  if (bits < kFilled * (uint32_t)__builtin_popcount(slots) || __builtin_popcountll(next) < 48)
    return false;
  const int64_t N = G.N;
  const BoxNbr<2> nb = row_nbr<2>(G, i);
  RowCtx<2> R;
  load_row<2>(G, A, i, A.tau[member(A, i)], R);
  double u2[NC];
  load_state<NC>(A.U1, N, i, u2);
  const double lam = 1.0 / G.lfac[i];
#pragma unroll 1
  for (int k = 0; k < 9; ++k) {
    const bool on = (nz >> k) & 1u;
    if (!__any(on)) continue;
    const int64_t j = on ? nb[k] : i, e = eidx<2>(k, i), et = eidx<2>(on ? tslot<2>(k) : k, j);
    const double la = A.lt2[e], lb = A.lt2[et];
    const bool both = on && ((A.nzm[j] >> tslot<2>(k)) & 1u);
    PIn<2> x;
    gather_P<2>(G, A, e, j, nb.mass(k), x);
    double P[NC];
    make_P<2>(R, x, P);
    const double w = both ? lam * fmin(la, lb) : 0.0;
#pragma unroll
    for (int q = 0; q < NC; ++q) u2[q] += on ? w * P[q] : 0.0;
  }
  if (nz) finish<2>(G, A, i, u2);
  return true;
}

template <typename LT>
__global__ __launch_bounds__(kWide) void k_fin_rows(DevGraphT<LT> G, StageArgsT<LT> A) {
  const uint32_t ns = spec_groups(G), tid = threadIdx.x;
  const int lane = tid & 63;
  if (A.keep && blockIdx.x == 0 && tid < 128) {
    // root entries of both passes: wave p sums pass p + 1's counts
    const uint32_t p = tid >> 6;
    uint32_t c = 0;
    for (uint32_t t = lane; t < gridDim.x; t += 64) c += A.q2[kRootWords + 2 * t + p];
#pragma unroll
    for (int d = 32; d > 0; d >>= 1) c += __shfl_xor(c, d);
    if (lane == 0) A.qcnt[p] = c;
  }
  wave_rows(G, A, ns, [&](uint32_t row, bool ok) __attribute__((always_inline)) {
    fin_pairs<LT>(G, A, row, lane & 7, lane & ~7, ok);
  }, [&](uint32_t row, bool ok) __attribute__((always_inline)) {
    return fin_dense<LT>(G, A, row, ok);
  });
}

// ---------------------------------------------------------------------------
// 3D, two passes (launch path): k_lim_first as in 2D, then the limited entries
// only.  In a shock tube four rows of five have some limited pair, but only a
// tenth of the entries: a wave takes a slice of 64 rows, collects their limited
// entries and gives each a lane, as many whole rows at a time as have at most
// 64 of them.  A lane forms its entry's P_ij and P_ji, runs both searches
// (roots included), and the rows' lanes subtract what pass 1 takes from
// U^L + lambda sum P; then the pass-2 search of the same entries follows, and
// rows without a pass-2 part are finished.  k_fin_entries adds that part of
// the others the same way.  Against three sweeps over all entries that
// gathered slot by slot, two root kernels and a final sweep (FP64, limiter and
// final update of a stage): 6.48 -> 3.95 ms at 192^3, 2.01 -> 1.13 ms at 128^3,
// and 0.56 -> 0.27 ms at 101 x 67 x 83 with FP32 coefficients.  k_lim_first
// (1.25 ms at 192^3) is bound by arithmetic and load latency at 3 waves per
// SIMD (held to 4 it spills: 1.4 times the time).  k_lim_entries (1.88 ms) spends
// a quarter of it in the root finder, the rest on each group's chain of gathers; so
// does k_fin_entries (0.82 ms).  3 waves per SIMD, since at 4 the former spills and
// is slower by 2%.
__device__ __forceinline__ void wave_sync() {
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  __builtin_amdgcn_wave_barrier();
}

// Counters of entries with a root (KEEP): kRootCnt of each pass, 8 words apart
// in A.q2, cleared by k_lo and summed by k_fin_entries (a single one would
// serialise the workgroups).
constexpr uint32_t kRootCnt = 64;

// Neighbour and m_ij of entry k of an interior row, by offset.
struct Entry3 {
  int32_t j;
  double m;
};
__device__ __forceinline__ Entry3 interior_entry(const BoxGeom *geo, int64_t i, int k) {
  const int dx = k % 3 - 1, dy = (k / 3) % 3 - 1, dz = k / 9 - 1;
  const int n0 = geo_ld(&geo->n[0]), n1 = geo_ld(&geo->n[1]);
  Entry3 e;
  e.j = (int32_t)i + dx + n0 * (dy + n1 * dz);
  e.m = geo->im[(dx ? 1 : 0) | (dy ? 2 : 0) | (dz ? 4 : 0)];
  return e;
}

// Slots of row i at which the neighbour's mask holds the pair (i, j): slot k
// is the neighbour's slot 26 - k.
__device__ __forceinline__ uint32_t line_bits(const BoxGeom *geo, const uint32_t *mask,
                                              int64_t r0, int64_t N, uint32_t tid) {
  const int64_t n0 = geo_ld(&geo->n[0]), n01 = n0 * geo_ld(&geo->n[1]);
  const bool edge = ((tid + 1) & 63) < 2;
  uint32_t bits = 0;
  static_for<0, 9>([&](auto line) __attribute__((always_inline)) {
    constexpr int ln = decltype(line)::value, dy = ln % 3 - 1, dz = ln / 3 - 1;
    const Line L = make_line(r0, dy * n0 + dz * n01, N, tid);
    const uint32_t mc = line_ld(mask, L.b, L.c);
    uint32_t mh = 0;
    if (edge) mh = line_ld(mask, L.b, L.h);
    bits |= ((from_left(mh, mc) >> (26 - 3 * ln)) & 1u) << (3 * ln);
    if constexpr (ln != 4) bits |= ((mc >> (25 - 3 * ln)) & 1u) << (3 * ln + 1);
    bits |= ((from_right(mh, mc) >> (24 - 3 * ln)) & 1u) << (3 * ln + 2);
  });
  return bits;
}
template <typename LT>
__device__ __forceinline__ uint32_t listed_bits(const DevGraphT<LT> &G, const uint32_t *mask,
                                                int64_t i) {
  const BoxNbr<3> nb = row_nbr<3>(G, i);
  uint32_t bits = 0;
#pragma unroll 1
  for (int k = 0; k < 27; ++k) {
    const int32_t j = nb[k];
    if (k != 13 && j >= 0) bits |= ((mask[j] >> (26 - k)) & 1u) << k;
  }
  return bits;
}

// Off-diagonal slots of row i.
template <typename LT>
__device__ __forceinline__ uint32_t listed_slots(const DevGraphT<LT> &G, int64_t i) {
  const BoxNbr<3> nb = row_nbr<3>(G, i);
  uint32_t bits = 0;
#pragma unroll 1
  for (int k = 0; k < 27; ++k)
    if (k != 13 && nb[k] >= 0) bits |= 1u << k;
  return bits;
}
constexpr uint32_t kAnew = 0x8000u;  // bit of an entry's id (see share_taken)

template <int SEV, bool KEEP, typename LT>
__global__ __launch_bounds__(kBlock) __attribute__((amdgpu_waves_per_eu(3, 3))) void
k_lim_entries(DevGraphT<LT> G, StageArgsT<LT> A, Gas g) {
#pragma clang fp contract(off)
  constexpr int NC = 5, NW = kBlock / 64;
  __shared__ double vals[NW][NC][64], nbw[NW][11][64];
  __shared__ float taken[NW][64];
  __shared__ uint32_t nzs[NW][64];
  __shared__ uint16_t ids[NW][64];
  const int64_t N = G.N;
  const uint32_t tid = threadIdx.x, lane = tid & 63;
  const uint32_t wv = __builtin_amdgcn_readfirstlane(tid >> 6);
  const uint32_t ns = spec_slices(G.nsrow);
  const bool front = blockIdx.x < ns;
  int64_t i;
  bool act;
  uint32_t lim = 0;
  const BoxGeom *geo = G.geo;
  if (front) {
    const int t = (int)(blockIdx.x * kBlock + tid);
    act = t < G.nsrow;
    i = G.srow[min(t, G.nsrow - 1)];
    lim = A.lim[i] | listed_bits(G, A.lim, i);
  } else {
    const uint32_t blk = blockIdx.x - ns;
    const int64_t r0 = (int64_t)blk * kBlock;
    geo = block_geo(G, blk);
    act = line_row(G, r0 + tid);
    i = min(r0 + (int64_t)tid, N - 1);
    lim = A.lim[i] |
          line_bits(geo, A.lim, r0, N, tid);
  }
  if (!act) lim = 0;
  const int mem = member(A, i);
  double u1[NC];
  load_state<NC>(A.U1, N, i, u1);
  nzs[wv][lane] = 0;
  uint32_t cnt = (uint32_t)__builtin_popcount(lim);
  uint32_t upto = wave_scan(cnt, lane);
  uint32_t start = 0, base = 0, n1 = 0, n2 = 0;
  uint32_t anew = 0;  // kAnew: this row is summed from U^L, all entries listed
  while (start < 64) {
    // rows start .. end-1: their entries fill at most the wave's lanes
    const uint64_t fits = __ballot(lane >= start && upto - base <= 64);
    const uint32_t end = start + (uint32_t)__builtin_popcountll(fits);
    const uint32_t total = (uint32_t)__builtin_amdgcn_readlane((int)upto, (int)end - 1) - base;
    const bool mine = lane >= start && lane < end;
    const uint32_t p0 = upto - cnt - base;  // this row's first entry
    if (total) {
      wave_sync();
      if (mine) {
        uint32_t m = lim;
        for (uint32_t p = p0; m; ++p) {
          ids[wv][p] = (uint16_t)(anew | lane << 5 | (uint32_t)__builtin_ctz(m));
          m &= m - 1;
        }
      }
      wave_sync();
      const bool ok = lane < total;
      const uint32_t id = ids[wv][ok ? lane : 0];
      const int r = (int)(id >> 5 & 63u), k = (int)(id & 31u);
      const int64_t ir = __shfl((int)i, r);
      const double tau = A.tau[__shfl(mem, r)];
      Entry3 en;
      if (front) {
        const BoxNbr<3> nb = row_nbr<3>(G, ir);
        en.j = nb[k];
        en.m = nb.mass(k);
      } else {
        en = interior_entry(geo, ir, k);
      }
      const int64_t e = eidx<3>(k, ir);
      const double lam = 1.0 / G.lfac[ir];
      double P[NC], own, rj = 1.0, ul[NC];
      Bounds b;
      uint32_t pend = 0;
      {
        RowCtx<3> R;
        PIn<3> x;
        double uj[NC], Pj[NC];
        load_row<3>(G, A, ir, tau, R);
        gather_P<3>(G, A, e, en.j, en.m, x);
        load_state<NC>(A.UL, N, ir, ul);
        load_state<NC>(A.UL, N, en.j, uj);
        b = load_bounds(A, N, ir);
        const Bounds bj = load_bounds(A, N, en.j);
        make_P_both<3>(R, x, tau * G.crm[en.j], P, Pj);
        if (ok && limit_fast<3, SEV>(g, uj, Pj, bj, &rj)) {
          pend = 2;
#pragma unroll
          for (int q = 0; q < NC; ++q) {
            nbw[wv][q][lane] = uj[q];
            nbw[wv][NC + q][lane] = Pj[q];
          }
          nbw[wv][2 * NC][lane] = bj.pmin;
        }
      }
      double s1 = 1.0, l2 = 0.0;
      bool again = false;
      const uint32_t n1_before = n1;
#pragma unroll 1
      for (int pass = 0; pass < 2; ++pass) {
        double r0 = pass ? 0.0 : 1.0;
        const bool slow = ok && s1 != 0.0 && limit_fast<3, SEV>(g, ul, P, b, &r0);
        if (slow) pend |= 1;
        if (KEEP) (pass ? n2 : n1) += (uint32_t)__builtin_popcountll(__ballot(slow));
#pragma unroll 1
        while (__any(pend)) {  // the root finder, for every lane's next search
          const bool nbr = pend == 2;
          double us[NC], Ps[NC], pm = b.pmin;
#pragma unroll
          for (int q = 0; q < NC; ++q) {
            us[q] = ul[q];
            Ps[q] = P[q];
          }
          if (nbr) {
#pragma unroll
            for (int q = 0; q < NC; ++q) {
              us[q] = nbw[wv][q][lane];
              Ps[q] = nbw[wv][NC + q][lane];
            }
            pm = nbw[wv][2 * NC][lane];
          }
          if (pend) {
            const double p2 = pm * pm;
            const double lr = (double)to_lt_down<LT>(nbr ? rj : r0);
            const double x = entropy_root_fast<3, SEV>(g, us, Ps, lr, pm, p2 * p2 * pm);
            if (nbr) rj = x;
            else r0 = x;
            pend &= pend - 1;
          }
        }
        if (pass == 0) {
          own = (double)to_lt_down<LT>(r0);
          const double l = fmin(own, (double)to_lt_down<LT>(rj));
          s1 = 1.0 - l;
          const double ls = lam * (id & kAnew ? l : s1);
          double t[NC];
#pragma unroll
          for (int q = 0; q < NC; ++q) vals[wv][q][lane] = t[q] = ls * P[q];
          const float share = ls != 0.0 ? share_taken<3>(ul, t) : 0.0f;
          wave_sync();
          if (__any(share > kMostTaken / 32)) {  // (26 smaller ones: below the limit)
            taken[wv][lane] = share;
            wave_sync();
            float most = 0.0f;
            if (mine && !anew)
              for (uint32_t p = p0; p < p0 + cnt; ++p) most += taken[wv][p];
            again = most > kMostTaken;
            if (__any(again)) break;
          }
          if (mine) {  // in slot order
            double sub[NC];
#pragma unroll
            for (int q = 0; q < NC; ++q) sub[q] = anew ? u1[q] : 0.0;
            for (uint32_t p = p0; p < p0 + cnt; ++p)
#pragma unroll
              for (int q = 0; q < NC; ++q) sub[q] += vals[wv][q][p];
#pragma unroll
            for (int q = 0; q < NC; ++q) u1[q] = anew ? sub[q] : u1[q] - sub[q];
          }
          wave_sync();
          if (mine) {
#pragma unroll
            for (int q = 0; q < NC; ++q) vals[wv][q][lane] = u1[q];
          }
          wave_sync();
#pragma unroll
          for (int q = 0; q < NC; ++q) {
            ul[q] = vals[wv][q][r];
            P[q] *= s1;
          }
        } else {
          l2 = r0 * s1;
        }
      }
      if (__any(again)) {  // these rows once more, with all their entries
        if (again) {
          anew = kAnew;
          lim = front ? listed_slots(G, i) : 0x7ffdfffu;
          load_state<NC>(A.UL, N, i, u1);
        }
        n1 = n1_before;
        cnt = (uint32_t)__builtin_popcount(lim);
        upto = wave_scan(cnt, lane);
        base = start ? (uint32_t)__builtin_amdgcn_readlane((int)upto, (int)start - 1) : 0;
        continue;
      }
      const LT sv = to_lt_down<LT>(l2);
      if (ok) {
        if constexpr (KEEP) A.lt1[e] = (LT)own;
        if (KEEP || sv != LT(0)) A.lt2[e] = sv;
        if (sv != LT(0)) atomicOr(&nzs[wv][r], 1u << k);
      }
    }
    start = end;
    base += total;
  }
  wave_sync();
  const uint32_t nz = nzs[wv][lane];
  if (act) {
    A.nzm[i] = nz;
    if (KEEP || nz) store_state<NC>(A.U1, N, i, u1);
    if (!nz) finish<3>(G, A, i, u1);
  }
  if constexpr (KEEP) {
    if (lane == 0 && (n1 | n2)) {
      uint32_t *c = A.q2 + 8 * (blockIdx.x % kRootCnt);
      atomicAdd(c, n1);
      atomicAdd(c + 8 * kRootCnt, n2);
    }
  }
}

// U = U^(1) + lambda_i sum l' (1 - l) P of the rows with a pass-2 part: their
// entries' products by lanes as in k_lim_entries, added in slot order.
template <typename LT>
__global__ __launch_bounds__(kBlock) void k_fin_entries(DevGraphT<LT> G, StageArgsT<LT> A) {
#pragma clang fp contract(off)
  constexpr int NC = 5, NW = kBlock / 64;
  __shared__ double vals[NW][NC][64];
  __shared__ uint16_t ids[NW][64];
  const int64_t N = G.N;
  const uint32_t tid = threadIdx.x, lane = tid & 63;
  const uint32_t wv = __builtin_amdgcn_readfirstlane(tid >> 6);
  const uint32_t ns = spec_slices(G.nsrow);
  const bool front = blockIdx.x < ns;
  if (A.keep && blockIdx.x == 0 && tid < 2 * kRootCnt) {
    uint32_t c = A.q2[8 * tid];
#pragma unroll
    for (int d = 32; d > 0; d >>= 1) c += __shfl_xor(c, d);
    if (lane == 0) A.qcnt[wv] = c;
  }
  int64_t i;
  bool act;
  uint32_t bits;  // (a product that its row did not store is 0: its bit is clear)
  const BoxGeom *geo = G.geo;
  if (front) {
    const int t = (int)(blockIdx.x * kBlock + tid);
    act = t < G.nsrow;
    i = G.srow[min(t, G.nsrow - 1)];
    bits = listed_bits(G, A.nzm, i);
  } else {
    const uint32_t blk = blockIdx.x - ns;
    const int64_t r0 = (int64_t)blk * kBlock;
    geo = block_geo(G, blk);
    act = line_row(G, r0 + tid);
    i = min(r0 + (int64_t)tid, N - 1);
    bits = line_bits(geo, A.nzm, r0, N, tid);
  }
  const uint32_t own = act ? A.nzm[i] : 0u, nz = own & bits;
  if (!__any(own)) return;
  const int mem = member(A, i);
  double u2[NC];
  load_state<NC>(A.U1, N, i, u2);
  const uint32_t cnt = (uint32_t)__builtin_popcount(nz);
  const uint32_t upto = wave_scan(cnt, lane);
  uint32_t start = 0, base = 0;
  while (start < 64) {
    const uint64_t fits = __ballot(lane >= start && upto - base <= 64);
    const uint32_t end = start + (uint32_t)__builtin_popcountll(fits);
    const uint32_t total = (uint32_t)__builtin_amdgcn_readlane((int)upto, (int)end - 1) - base;
    const bool mine = lane >= start && lane < end;
    const uint32_t p0 = upto - cnt - base;
    if (total) {
      wave_sync();
      if (mine) {
        uint32_t m = nz;
        for (uint32_t p = p0; m; ++p) {
          ids[wv][p] = (uint16_t)(lane << 5 | (uint32_t)__builtin_ctz(m));
          m &= m - 1;
        }
      }
      wave_sync();
      const bool ok = lane < total;
      const uint32_t id = ids[wv][ok ? lane : 0];
      const int r = (int)(id >> 5), k = (int)(id & 31u);
      const int64_t ir = __shfl((int)i, r);
      const double tau = A.tau[__shfl(mem, r)];
      Entry3 en;
      if (front) {
        const BoxNbr<3> nb = row_nbr<3>(G, ir);
        en.j = nb[k];
        en.m = nb.mass(k);
      } else {
        en = interior_entry(geo, ir, k);
      }
      const int64_t e = eidx<3>(k, ir), et = eidx<3>(tslot<3>(k), en.j);
      const double la = A.lt2[e], lb = A.lt2[et];
      RowCtx<3> R;
      PIn<3> x;
      load_row<3>(G, A, ir, tau, R);
      gather_P<3>(G, A, e, en.j, en.m, x);
      const double w = 1.0 / G.lfac[ir] * fmin(la, lb);
      double P[NC];
      make_P<3>(R, x, P);
#pragma unroll
      for (int q = 0; q < NC; ++q) vals[wv][q][lane] = w * P[q];
      wave_sync();
      if (mine)
        for (uint32_t p = p0; p < p0 + cnt; ++p)
#pragma unroll
          for (int q = 0; q < NC; ++q) u2[q] += vals[wv][q][p];
    }
    start = end;
    base += total;
  }
  if (own) finish<3>(G, A, i, u2);
}

// Pass-2 line search on (1 - l_ij) P_ij from U^(1) (stored by lim2_row).
template <int DIM, int SEV, typename LT>
__device__ __forceinline__ void lim2b_row(const DevGraphT<LT> &G, const StageArgsT<LT> &A,
                                          const Gas &g, uint32_t blk, int64_t i) {
  using C = Cfg<DIM, NS_CH_LIM2>;
  constexpr int NC = C::NC;
  const int64_t N = G.N;
  if (i >= N) return;
  const LT *__restrict__ lt1 = A.lt1;
  LT *__restrict__ lt2 = A.lt2;
  BoxNbr<DIM> jv = block_nbr<DIM>(G, blk, i);
  RowCtx<DIM> R;
  load_row<DIM>(G, A, i, A.tau[member(A, i)], R);
  double u1[NC];
  load_state<NC>(A.U1, N, i, u1);
  const Bounds b = load_bounds(A, N, i);
  uint32_t slow = 0;
#pragma unroll
  for (int ch = 0; ch < C::NCH; ++ch) {
    jv.fence();
    double la[C::CH], lb[C::CH];
    int32_t jc[C::CH];
#pragma unroll
    for (int kk = 0; kk < C::CH; ++kk) {
      const int k = ch * C::CH + kk;
      const int64_t e = eidx<DIM>(k, i);
      jc[kk] = jv[k];
      if (k == C::W / 2) continue;  // the diagonal
      const int64_t js = jc[kk] >= 0 ? jc[kk] : i;
      la[kk] = lt1[e];
      lb[kk] = lt1[eidx<DIM>(tslot<DIM>(k), js)];
    }
#pragma unroll
    for (int kk = 0; kk < C::CH; ++kk) {
      const int k = ch * C::CH + kk;
      if (jc[kk] < 0 || jc[kk] == i) continue;
      double P[NC], l2 = 0.0;
      const double s1 = 1.0 - fmin(la[kk], lb[kk]);
      // else the stored product is 0, and P_ij's inputs are
      // not gathered
      if (s1 != 0.0) {
        PIn<DIM> x;
        gather_P<DIM>(G, A, eidx<DIM>(k, i), jc[kk], jv.mass(k), x);
        make_P<DIM>(R, x, P);
#pragma unroll
        for (int q = 0; q < NC; ++q) P[q] *= s1;
        if (limit_fast<DIM, SEV>(g, u1, P, b, &l2)) slow |= 1u << k;
        else l2 *= s1;
      }
      st_once(&lt2[eidx<DIM>(k, i)], to_lt_down<LT>(l2));
    }
  }
  if (slow) {
    uint32_t *__restrict__ q2 = A.q2;
    uint32_t t = atomicAdd(&A.qcnt[1], (uint32_t)__builtin_popcount(slow));
    while (slow) {
      const int k = __builtin_ctz(slow);
      slow &= slow - 1;
      q2[t++] = (uint32_t)eidx<DIM>(k, i);
    }
  }
}

// Row of a sliced-ELL edge index (inverse of eidx in the row).
template <int DIM>
__device__ __forceinline__ int64_t edge_row(int64_t e) {
  constexpr int W = DIM == 2 ? 9 : 27;
  return ((e >> 6) / W) * 64 + (e & 63);
}

// Roots of the entropy bound for the work list of limiter pass PASS (1 or 2):
// one lane per listed entry, grid-stride over the list, so the rare root
// finder runs at full occupancy instead of stalling a row sweep's wavefront.
// The line search's density limit l_rho was stored in lt by the sweep.
// List entries start, start + stride, ... below the list length.
template <int DIM, int PASS, int SEV, typename LT>
__device__ __forceinline__ void root_range(const DevGraphT<LT> &G, const StageArgsT<LT> &A,
                                           const Gas &g, uint32_t start, uint32_t stride) {
  constexpr int NC = DIM + 2;
  const int64_t N = G.N;
  const uint32_t n = A.qcnt[PASS - 1];
  const uint32_t *__restrict__ q = PASS == 2 ? A.q2 : A.q;
  LT *__restrict__ lt = PASS == 1 ? A.lt1 : A.lt2;
  for (uint32_t t = start; t < n; t += stride) {
    const int64_t e = q[t];
    const int64_t i = edge_row<DIM>(e);
    const int k = (int)((e >> 6) % (DIM == 2 ? 9 : 27));
    const BoxNbr<DIM> nb = row_nbr<DIM>(G, i);
    const int32_t j = nb[k];
    RowCtx<DIM> R;
    load_row<DIM>(G, A, i, A.tau[member(A, i)], R);
    double u[NC], P[NC];
    load_state<NC>(PASS == 1 ? A.UL : A.U1, N, i, u);
    const Bounds b = load_bounds(A, N, i);
    compute_P<DIM>(G, A, R, e, j, nb.mass(k), P);
    double s1 = 1.0;
    if constexpr (PASS == 2) {
      s1 = 1.0 - fmin(A.lt1[e], A.lt1[eidx<DIM>(tslot<DIM>(k), j)]);
#pragma unroll
      for (int c = 0; c < NC; ++c) P[c] *= s1;
    }
    const double l = entropy_root_fast<DIM, SEV>(g, u, P, lt[e], b.pmin, b.pmin5);
    lt[e] = to_lt_down<LT>(PASS == 2 ? l * s1 : l);
  }
}

template <int DIM, int SEV, typename LT>
__global__ __launch_bounds__(kBlock) void k_root(DevGraphT<LT> G, StageArgsT<LT> A, Gas g) {
  root_range<DIM, 1, SEV, LT>(G, A, g, blockIdx.x * kBlock + threadIdx.x,
                              gridDim.x * kBlock);
}

template <int DIM, typename LT>
__device__ __forceinline__ void fin_row(const DevGraphT<LT> &G, const StageArgsT<LT> &A,
                                        const Gas &g, uint32_t blk, int64_t i) {
#pragma clang fp contract(off)  // the same bits in every kernel
  using C = Cfg<DIM, NS_CH_FIN>;
  constexpr int NC = C::NC;
  const int64_t N = G.N;
  if (i >= N) return;
  const LT *__restrict__ lt2 = A.lt2;
  BoxNbr<DIM> jv = block_nbr<DIM>(G, blk, i);
  double u2[NC];
  load_state<NC>(A.U1, N, i, u2);
  // lt2 holds l~'_ij (1 - l_ij) with l_ij the symmetric pass-1 limiter;
  // (1 - l_ij) >= 0 and equal at ij and ji, and rounding is monotone, so the
  // smaller stored product is min(l~'_ij, l~'_ji) (1 - l_ij) itself.  It is
  // 0 wherever pass 1 took the whole P_ij (most entries away from shocks).
  // 2D: only rows with such an entry, a few in a hundred, load their own
  // data and the P_ij of those entries.
  // 3D, where most rows behind the shock have such entries, keeps one
  // unrolled pass (the entry-by-entry loop doubled the sweep's time there).
  if constexpr (DIM == 3) {
    RowCtx<DIM> R;
    load_row<DIM>(G, A, i, A.tau[member(A, i)], R);
    const double lam = 1.0 / G.lfac[i];
#pragma unroll
    for (int ch = 0; ch < C::NCH; ++ch) {
      jv.fence();
      double l2a[C::CH], l2b[C::CH];
      int32_t jc[C::CH];
#pragma unroll
      for (int kk = 0; kk < C::CH; ++kk) {
        const int k = ch * C::CH + kk;
        const int64_t e = eidx<DIM>(k, i);
        jc[kk] = jv[k];
        if (k == C::W / 2) continue;  // the diagonal
        const int64_t js = jc[kk] >= 0 ? jc[kk] : i;
        l2a[kk] = lt2[e];
        l2b[kk] = lt2[eidx<DIM>(tslot<DIM>(k), js)];
      }
#pragma unroll
      for (int kk = 0; kk < C::CH; ++kk) {
        const int k = ch * C::CH + kk;
        if (jc[kk] < 0 || jc[kk] == i) continue;
        const double w = lam * fmin(l2a[kk], l2b[kk]);
        if (w == 0.0) continue;  // no contribution, no gather
        PIn<DIM> x;
        gather_P<DIM>(G, A, eidx<DIM>(k, i), jc[kk], jv.mass(k), x);
        double P[NC];
        make_P<DIM>(R, x, P);
#pragma unroll
        for (int q = 0; q < NC; ++q) u2[q] += w * P[q];
      }
    }
    finish<DIM>(G, A, i, u2);
    return;
  }
  // the row's slots whose stored product may be nonzero, from k_lim2 (an
  // entry needs its own product nonzero)
  uint32_t nz = A.nzm[i];
  if (nz) {
    RowCtx<DIM> R;
    load_row<DIM>(G, A, i, A.tau[member(A, i)], R);
    const double lam = 1.0 / G.lfac[i];
    while (nz) {  // in slot order, as the sum over the row
      const int k = __builtin_ctz(nz);
      nz &= nz - 1;
      const int32_t j = jv[k];
      const double la = lt2[eidx<DIM>(k, i)], lb = lt2[eidx<DIM>(tslot<DIM>(k), j)];
      const double w = lam * fmin(la, lb);
      if (w == 0.0) continue;
      PIn<DIM> x;
      gather_P<DIM>(G, A, eidx<DIM>(k, i), j, jv.mass(k), x);
      double P[NC];
      make_P<DIM>(R, x, P);
#pragma unroll
      for (int q = 0; q < NC; ++q) u2[q] += w * P[q];
    }
  }
  finish<DIM>(G, A, i, u2);
}

template <int DIM, typename LT>
__global__ __launch_bounds__(kBlock) void k_combine_low(DevGraphT<LT> G, StageArgsT<LT> A) {
  constexpr int NC = DIM + 2;
  const int64_t i = row_id();
  if (i >= G.N) return;
  double u[NC];
  load_state<NC>(A.UL, G.N, i, u);
  finish<DIM>(G, A, i, u);
}

// Slip projection of list entry t (entries below end).
template <int DIM>
__device__ __forceinline__ void slip_one(int t, int end, const int32_t *__restrict__ idx,
                                         const double *__restrict__ nrm, int stride,
                                         int64_t N, double *__restrict__ U) {
  if (t >= end) return;
  const int64_t i = idx[t];
  double n[DIM], mn = 0.0;
#pragma unroll
  for (int k = 0; k < DIM; ++k) {
    n[k] = nrm[(int64_t)k * stride + t];
    mn = fma(U[node_at(DIM + 2, 1 + k, i, N)], n[k], mn);
  }
#pragma unroll
  for (int k = 0; k < DIM; ++k) U[node_at(DIM + 2, 1 + k, i, N)] -= mn * n[k];
}

template <int DIM>
__global__ __launch_bounds__(kBlock) void k_slip(int nslip,
                                                 const int32_t *__restrict__ idx,
                                                 const double *__restrict__ nrm,
                                                 int stride, int64_t N,
                                                 double *__restrict__ U) {
  slip_one<DIM>(blockIdx.x * kBlock + threadIdx.x, nslip, idx, nrm, stride, N, U);
}

__global__ __launch_bounds__(kBlock) void k_copy(const double2 *__restrict__ src,
                                                 double2 *__restrict__ dst,
                                                 int64_t n16) {
  const int64_t t = plain_id();
  if (t < n16) dst[t] = src[t];
}

__global__ __launch_bounds__(kBlock) void k_copy8(const double *__restrict__ src,
                                                  double *__restrict__ dst,
                                                  int64_t n8) {
  const int64_t t = plain_id();
  if (t < n8) dst[t] = src[t];
}

// Component-major rows (component c of row t at c*ns + t) to and from rows
// first .. first+count-1 of a node vector of N rows (node_layout.hpp).
template <int NC>
__global__ __launch_bounds__(kBlock) void k_nodes_from_cm(const double *__restrict__ src,
                                                          int64_t ns, double *__restrict__ dst,
                                                          int64_t N, int64_t first,
                                                          int64_t count) {
  const int64_t t = plain_id();
  if (t >= count) return;
#pragma unroll
  for (int c = 0; c < NC; ++c) dst[node_at(NC, c, first + t, N)] = src[c * ns + t];
}

template <int NC>
__global__ __launch_bounds__(kBlock) void k_nodes_to_cm(const double *__restrict__ src,
                                                        int64_t N, int64_t first,
                                                        int64_t count, double *__restrict__ dst,
                                                        int64_t ns) {
  const int64_t t = plain_id();
  if (t >= count) return;
#pragma unroll
  for (int c = 0; c < NC; ++c) dst[c * ns + t] = src[node_at(NC, c, first + t, N)];
}

__global__ void k_set_scalar(double *p, double v, int n) {
  const int t = blockIdx.x * 64 + threadIdx.x;
  if (t < n) p[t] = v;
}

__global__ void k_add_scalar(double *acc, const double *v, int n) {
  const int t = blockIdx.x * 64 + threadIdx.x;
  if (t < n) acc[t] += v[t];
}

__global__ void k_clear_flags(int *flags, int n) {
  const int t = blockIdx.x * 64 + threadIdx.x;
  if (t < 4 * n) flags[t] = (t & 3) == 2 ? INT_MAX : 0;
}

template <int DIM>
__global__ __launch_bounds__(kBlock) void k_check_state(int64_t N,
                                                        const double *__restrict__ U,
                                                        int *__restrict__ flags) {
  constexpr int NC = DIM + 2;
  const int64_t i = plain_id();
  if (i >= N) return;
  double u[NC];
  load_state<NC>(U, N, i, u);
  bool ok = u[0] > 0.0;
  double m2 = 0.0;
#pragma unroll
  for (int k = 0; k < DIM; ++k) m2 += u[1 + k] * u[1 + k];
  const double eps = u[NC - 1] - 0.5 * m2 / u[0];
  ok = ok && eps > 0.0 && isfinite(eps);
#pragma unroll
  for (int q = 0; q < NC; ++q) ok = ok && isfinite(u[q]);
  if (!ok) {
    flags[1] = 1;
    atomicMin(&flags[2], (int)i);
  }
}

// ---------------------------------------------------------------------------
// Diagnostics (ns_stats): minimum density and internal energy of a state and
// the limiter activity of the last stage.  Rows are strided over a fixed grid
// so that the partial results need kStatsParts slots whatever N is.
struct MinArg {
  double v;
  int64_t i;
};
__device__ __forceinline__ MinArg min_arg(MinArg a, MinArg b) {
  // smaller value, ties to the smaller index (NaN never wins)
  return (b.v < a.v || (b.v == a.v && b.i < a.i)) ? b : a;
}
__device__ __forceinline__ MinArg shfl_min_arg(MinArg a, int off) {
  MinArg b;
  b.v = __shfl_xor(a.v, off);
  b.i = __shfl_xor(a.i, off);
  return min_arg(a, b);
}

// Block reduction of the stats tuple; thread 0 holds the result.
__device__ __forceinline__ void block_stats(MinArg &r, MinArg &e, double &c0, double &c1,
                                            double &c2) {
  __shared__ MinArg sr[kBlock / 64], se[kBlock / 64];
  __shared__ double sc[3][kBlock / 64];
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) {
    r = shfl_min_arg(r, off);
    e = shfl_min_arg(e, off);
    c0 += __shfl_xor(c0, off);
    c1 += __shfl_xor(c1, off);
    c2 += __shfl_xor(c2, off);
  }
  const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
  if (lane == 0) {
    sr[wid] = r; se[wid] = e; sc[0][wid] = c0; sc[1][wid] = c1; sc[2][wid] = c2;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    for (int w = 1; w < kBlock / 64; ++w) {
      r = min_arg(r, sr[w]);
      e = min_arg(e, se[w]);
      c0 += sc[0][w]; c1 += sc[1][w]; c2 += sc[2][w];
    }
  }
}

// part[b*7 + ...] = min rho, its node, min eps, its node, off-diagonal
// entries, entries with l < 1 after pass 1, entries with l + l'(1 - l) < 1
// after pass 2 (counts as doubles: exact below 2^53).
template <int DIM, typename LT>
__global__ __launch_bounds__(kBlock) void k_stats_partial(DevGraphT<LT> G,
                                                          const double *__restrict__ U,
                                                          const LT *__restrict__ lt1,
                                                          const LT *__restrict__ lt2,
                                                          int mode, double *__restrict__ part) {
  constexpr int NC = DIM + 2, W = DIM == 2 ? 9 : 27;
  const int64_t N = G.N;
  MinArg r{INFINITY, INT64_MAX}, e{INFINITY, INT64_MAX};
  double cnt = 0.0, c1 = 0.0, c2 = 0.0;
  for (int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x; i < N;
       i += (int64_t)gridDim.x * kBlock) {
    double u[NC];
    load_state<NC>(U, N, i, u);
    double m2 = 0.0;
#pragma unroll
    for (int k = 0; k < DIM; ++k) m2 += u[1 + k] * u[1 + k];
    r = min_arg(r, MinArg{u[0], i});
    e = min_arg(e, MinArg{u[NC - 1] - 0.5 * m2 / u[0], i});
    const BoxNbr<DIM> nb = row_nbr<DIM>(G, i);
    for (int k = 0; k < W; ++k) {
      const int32_t j = nb[k];
      if (j < 0 || j == i) continue;
      cnt += 1.0;
      if (mode == 0) continue;
      const int64_t ea = eidx<DIM>(k, i), eb = eidx<DIM>(tslot<DIM>(k), j);
      const double l = fmin((double)lt1[ea], (double)lt1[eb]);
      if (l < 1.0) c1 += 1.0;
      if (mode == 2 && l + fmin((double)lt2[ea], (double)lt2[eb]) < 1.0) c2 += 1.0;
    }
  }
  block_stats(r, e, cnt, c1, c2);
  if (threadIdx.x == 0) {
    double *o = part + 7 * (int64_t)blockIdx.x;
    o[0] = r.v; o[1] = (double)r.i; o[2] = e.v; o[3] = (double)e.i;
    o[4] = cnt; o[5] = c1; o[6] = c2;
  }
}

__global__ __launch_bounds__(kBlock) void k_stats_final(const double *__restrict__ part,
                                                        int nparts, double *__restrict__ out) {
  MinArg r{INFINITY, INT64_MAX}, e{INFINITY, INT64_MAX};
  double c0 = 0.0, c1 = 0.0, c2 = 0.0;
  for (int b = threadIdx.x; b < nparts; b += kBlock) {
    const double *o = part + 7 * (int64_t)b;
    r = min_arg(r, MinArg{o[0], (int64_t)o[1]});
    e = min_arg(e, MinArg{o[2], (int64_t)o[3]});
    c0 += o[4]; c1 += o[5]; c2 += o[6];
  }
  block_stats(r, e, c0, c1, c2);
  if (threadIdx.x == 0) {
    out[0] = r.v; out[1] = (double)r.i; out[2] = e.v; out[3] = (double)e.i;
    out[4] = c0; out[5] = c1; out[6] = c2;
  }
}

// ---------------------------------------------------------------------------
// Persistent steps (PersistArgsT).  The workgroups take items in sequence
// order, so every item a workgroup waits for was taken earlier by a running
// workgroup, and the earliest unfinished item never waits: the launch makes
// progress whatever the number of resident workgroups.  A member's items of
// one phase depend only on that member's earlier phases, so members move
// through a stage independently.  Completion is published with a release at
// device scope (the stores of the item reach the device-coherent level
// before the counter moves) and a wait ends with an acquire (no stale cached
// copy is read afterwards).

// The two state buffers other than c, ascending (k = 0, 1).
__device__ __forceinline__ int other_buf(int c, int k) {
  return k == 0 ? (c == 0 ? 1 : 0) : (c == 2 ? 1 : 2);
}

// tau = cfl min over the member's row blocks; the time advanced grows by it
// (every thread of the workgroup calls it).
__device__ __forceinline__ void dt_final_member(const double *__restrict__ partial,
                                                int32_t b0, int32_t b1, double cfl,
                                                double *tau, double *tacc) {
  double v = INFINITY;
  for (int64_t b = b0 + threadIdx.x; b < b1; b += kBlock) v = fmin(v, partial[b]);
  v = block_min(v);
  if (threadIdx.x == 0) {
    const double t = cfl * v;
    *tau = t;
    *tacc += t;
  }
}

template <typename LT>
__device__ __forceinline__ bool persist_stopped(const PersistArgsT<LT> &P) {
  return __hip_atomic_load(P.stop, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != 0;
}

template <typename LT>
__device__ __forceinline__ void persist_raise(const PersistArgsT<LT> &P, int why) {
  atomicCAS(P.stop + 1, 0, why);
  atomicOr(P.stop + 2, 1 << why);
  __hip_atomic_store(P.stop, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

template <typename LT>
__device__ __forceinline__ bool persist_give_up(const PersistArgsT<LT> &P) {
  return P.give_up &&
         __hip_atomic_load(P.give_up, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM) != 0;
}

// Wave 0: waits until *ctr >= need (every lane polls the same word, so
// every branch is uniform over the wave) and returns the value it saw, or
// 0 if the launch stops first.  The counter is polled with relaxed loads (an
// acquire per poll would invalidate the caches the working workgroups read,
// on every poll of every waiting workgroup); the acquire follows once,
// after the wait.  The wait is bounded by wait_ticks of the wall clock and
// ends early when the launch is stopped or the give-up word is set (which
// then stops the launch).
template <typename LT>
__device__ uint32_t persist_wait(const PersistArgsT<LT> &P, const uint32_t *ctr,
                                 uint32_t need) {
  auto seen = [&] {
    return __builtin_amdgcn_readfirstlane(
        __hip_atomic_load(ctr, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT));
  };
  uint32_t v = seen();
  if (v < need) {
    const uint64_t t0 = wall_clock64();
    for (uint32_t it = 0;; ++it) {
      if (__builtin_amdgcn_readfirstlane(persist_stopped(P))) return 0;
      if ((it & 63u) == 0) {
        if (__builtin_amdgcn_readfirstlane(persist_give_up(P))) {
          if (threadIdx.x == 0) persist_raise(P, 2);
          return 0;
        }
        if (__builtin_amdgcn_readfirstlane(wall_clock64() - t0 >= P.wait_ticks)) {
          if (threadIdx.x == 0) persist_raise(P, 1);
          return 0;
        }
      }
      __builtin_amdgcn_s_sleep(8);
      v = seen();
      if (v >= need) break;
    }
  }
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
  return v;
}

// The control path (ticket, wait, publication) runs on wave 0 with
// conditions uniform over the wave, and only the atomics themselves on lane
// 0: a barrier reached under a condition the compiler takes as divergent
// within a wave -- e.g. thread 0 alone on both sides of the loop's back
// edge -- lets the structurizer nest the loop so that the other lanes repeat
// the barriers and the item on their own.
//
// Cache maintenance at device scope (write-back before a completion is
// published, invalidation after a wait) is paid per phase, not per item:
// a workgroup keeps its completed items pending and publishes them (one
// release, one counter update) only before it has to wait or moves to
// another member, and it skips the wait and the acquire when an earlier
// wait already saw the member's counter at or above the item's need.  A
// workgroup never waits while it holds pending items, so every pending item
// is published before anything can depend on it in a wait.
template <int DIM, int SEV, typename LT>
__global__ __launch_bounds__(kBlock) void k_persist(DevGraphT<LT> G, PersistArgsT<LT> P,
                                                    Gas g) {
  constexpr int W = DIM == 2 ? 9 : 27;
  __shared__ uint32_t s_item, s_seen;
  __shared__ int s_go;
  const int tid = threadIdx.x;
  const bool wave0 = __builtin_amdgcn_readfirstlane(tid) == 0;
  const PersistPlan &pl = P.plan;
  // uniform state, identical in every wave: the member and counter value of
  // the last acquire; the member and number of the pending completions
  int acq_m = -1, pend_m = -1;
  uint32_t acq_v = 0, pend_n = 0;
  auto publish = [&] {
    if (pend_n == 0) return;
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "agent");
    __syncthreads();
    if (wave0 && tid == 0)
      __hip_atomic_fetch_add(P.done + pend_m, pend_n, __ATOMIC_RELAXED,
                             __HIP_MEMORY_SCOPE_AGENT);
    pend_n = 0;
  };
  for (;;) {
    if (wave0) {
      int go = 0;
      uint32_t t = 0;
      if (!__builtin_amdgcn_readfirstlane(persist_stopped(P))) {
        uint32_t mine = 0;
        if (tid == 0) mine = atomicAdd(P.ticket, 1u);
        t = __builtin_amdgcn_readfirstlane(mine);
        if (t < P.items) {
          // the give-up word is also read every 16 items, so that it stops
          // a launch whose waits all end at once
          if ((t & 15u) == 0 && __builtin_amdgcn_readfirstlane(persist_give_up(P))) {
            if (tid == 0) persist_raise(P, 2);
          } else {
            go = 1;
          }
        }
      }
      if (tid == 0) {
        s_item = t;
        s_go = go;
      }
    }
    __syncthreads();
    if (!__builtin_amdgcn_readfirstlane(s_go)) {
      publish();
      return;
    }
    const uint32_t t = __builtin_amdgcn_readfirstlane(s_item);
    // item -> step, phase, member, item within the member's phase
    const uint32_t step = t / P.items_step;
    const uint32_t u = t - step * P.items_step;
    int p = 0;
    while (p + 1 < pl.nph && pl.off[p + 1] <= u) ++p;
    const int ph = pl.phase[p], st = pl.stage[p];
    const int kind = persist_kind(ph);
    uint32_t r = u - (uint32_t)pl.off[p];
    int m = 0;
    if (kind == PK_ONE) {
      m = (int)r;
      r = 0;
    } else {
      // (the member tables are read-only: scalar loads, uniform results)
      const int32_t *cum = kind == PK_ROW ? P.mblk : kind == PK_ROOT ? P.rblk : P.sblk;
      int lo = 0, hi = P.A.nmem;  // largest m with cum[m] <= r
      while (hi - lo > 1) {
        const int mid = (lo + hi) >> 1;
        if ((uint32_t)geo_ld(&cum[mid]) <= r) lo = mid;
        else hi = mid;
      }
      m = lo;
      r -= (uint32_t)geo_ld(&cum[m]);
    }
    const int32_t mb0 = geo_ld(&P.mblk[m]), mb1 = geo_ld(&P.mblk[m + 1]);
    const uint32_t nb = mb1 - mb0, nr = geo_ld(&P.rblk[m + 1]) - geo_ld(&P.rblk[m]),
                   ns = geo_ld(&P.sblk[m + 1]) - geo_ld(&P.sblk[m]);
    auto before = [&](int q) {
      return pl.pre[q][PK_ROW] * nb + pl.pre[q][PK_ROOT] * nr + pl.pre[q][PK_SLIP] * ns +
             (uint32_t)pl.pre[q][PK_ONE];
    };
    const uint32_t need = step * before(pl.nph) + before(p);
    if (m != pend_m) publish();
    if (m != acq_m || need > acq_v) {
      publish();
      if (wave0) {
        const uint32_t v = persist_wait(P, P.done + m, need);
        if (tid == 0) s_seen = v;
      }
      __syncthreads();  // (the acquire of wave 0 covers the workgroup's CU)
      const uint32_t v = __builtin_amdgcn_readfirstlane(s_seen);
      if (v < need) return;  // the launch stopped
      acq_m = m;
      acq_v = v;
    }
    // buffers of the stage (as the launch path rotates them)
    int c = P.cur;
    for (uint32_t k = 0; k < step; ++k) c = other_buf(c, 0);
    const int o1 = other_buf(c, 0), o2 = other_buf(c, 1);
    StageArgsT<LT> A = P.A;
    A.Un = P.S[c];
    if (st == 0) {
      A.U = P.S[c]; A.out = P.S[o1]; A.sa = 0.0; A.sb = 1.0; A.check_cfl = 0;
    } else if (st == 1) {
      A.U = P.S[o1]; A.out = P.S[o2]; A.sa = 0.75; A.sb = 0.25; A.check_cfl = 1;
    } else {
      A.U = P.S[o2]; A.out = P.S[o1]; A.sa = 1.0 / 3.0; A.sb = 2.0 / 3.0; A.check_cfl = 1;
    }
    // the member's own work lists: its slice of q and its two counters
    A.q = P.A.q + (int64_t)W * kBlock * mb0;
    A.q2 = A.q;  // root1 empties the list before lim2 fills it again
    A.qcnt = P.pcnt + 2 * m;
    const uint32_t blk = kind == PK_ROW ? (uint32_t)mb0 + r : 0u;
    const int64_t i = (int64_t)blk * kBlock + tid;
    switch (ph) {
      case PP_PRIM: prim_row<DIM>(G.N, A.U, A.aux, g, i); break;
      case PP_VISC:
        if (i < G.N)
          visc_row<DIM, 0, SEV, false, LT>(G, A.U, A.aux, A.d, A.alpha, g, block_nbr<DIM>(G, blk, i), i);
        break;
      case PP_DTP: dt_partial_blk<DIM, LT>(G, A.d, A.partial, blk, i); break;
      case PP_DTF:
        dt_final_member(A.partial, mb0, mb1, P.cfl, A.tau + m, P.tacc + m);
        break;
      case PP_LO:
        clear_lists(A, r == 0 && tid == 0);
        if (i < G.N) lo_row<DIM, false>(G, A, g, block_nbr<DIM>(G, blk, i), i);
        break;
      case PP_LIM1: lim1_row<DIM, SEV, LT>(G, A, g, blk, i); break;
      case PP_ROOT1: root_range<DIM, 1, SEV, LT>(G, A, g, r * kBlock + tid, nr * kBlock); break;
      case PP_LIM2: lim2_row<DIM, DIM == 2 ? 0 : 3, SEV, LT>(G, A, g, blk, i); break;
      case PP_LIM2B:
        if constexpr (DIM == 3) lim2b_row<DIM, SEV, LT>(G, A, g, blk, i);
        break;
      case PP_ROOT2: root_range<DIM, 2, SEV, LT>(G, A, g, r * kBlock + tid, nr * kBlock); break;
      case PP_FIN: fin_row<DIM, LT>(G, A, g, blk, i); break;
      case PP_SLIP:
        slip_one<DIM>(geo_ld(&P.mslip[m]) + (int)(r * kBlock) + tid, geo_ld(&P.mslip[m + 1]),
                      P.slip_idx, P.slip_n, P.nslip, G.N, A.out);
        break;
      default: break;
    }
    pend_m = m;
    ++pend_n;
  }
}

__global__ void k_persist_reset(uint32_t *done, uint32_t *pcnt, uint32_t *ticket, int *stop,
                                int nmem, int run_start) {
  const int t = blockIdx.x * 64 + threadIdx.x;
  if (t < nmem) done[t] = 0;
  if (t < 2 * nmem) pcnt[t] = 0;
  if (t == 0) {
    *ticket = 0;
    if (run_start) stop[2] = 0;
    stop[0] = stop[2] != 0;  // a launch after one that gave up stops at once
    stop[1] = 0;
  }
}

inline dim3 grid_for(int64_t n) { return dim3((unsigned)((n + kBlock - 1) / kBlock)); }

template <int DIM, int SEV, typename LT>
void stage_impl(const Gas &gas, const DevGraphT<LT> &G, const StageArgsT<LT> &A,
                int indicator, int limiter, int passes, bool auto_dt,
                double cfl, hipStream_t s, void (*before)(void *, const char *),
                void (*after)(void *), void *prof) {
  const dim3 grid = grid_for(G.N), block(kBlock);
  // sweeps along stencil lines: the listed rows' blocks in front
  const dim3 lgrid(grid.x + spec_blocks<DIM>(G));
#define NS_LAUNCH(name, ...)                                  \
  do {                                                        \
    before(prof, name);                                       \
    __VA_ARGS__;                                              \
    after(prof);                                              \
  } while (0)
  NS_LAUNCH("prim", hipLaunchKernelGGL(k_prim<DIM>, grid, block, 0, s, G.N, A.U, A.aux, gas,
                                       A.clear));
  bool f32 = false;
  if constexpr (SEV == 1 && sizeof(LT) == 4) {
    if (indicator == 0 && A.fp32_eval) {
      f32 = true;
      NS_LAUNCH("visc", hipLaunchKernelGGL((k_visc_f32<DIM, LT>), grid, block, 0, s, G, A.U,
                                           A.aux, A.d, A.alpha, gas));
    }
  }
  if (!f32) {
    auto visc = [&](auto ind) {
      constexpr int IND = decltype(ind)::value;
      if (G.byrow)
        NS_LAUNCH("visc", hipLaunchKernelGGL((k_visc_rows<DIM, IND, SEV, LT>), grid, block, 0, s,
                                             G, A.U, A.aux, A.d, A.alpha, gas));
      else
        NS_LAUNCH("visc", hipLaunchKernelGGL((k_visc<DIM, IND, SEV, LT>), lgrid, block, 0, s, G,
                                             A.U, A.aux, A.d, A.alpha, gas));
    };
    if (indicator == 0) visc(std::integral_constant<int, 0>{});
    else if (indicator == 1) visc(std::integral_constant<int, 1>{});
    else visc(std::integral_constant<int, 2>{});
  }
  if (auto_dt) {
    NS_LAUNCH("dt_partial", hipLaunchKernelGGL((k_dt_partial<DIM, LT>), grid, block, 0, s,
                                               G, A.d, A.partial));
    if (A.seg)
      NS_LAUNCH("dt_final", hipLaunchKernelGGL(k_dt_final_members, dim3((unsigned)A.nmem),
                                               dim3(1024), 0, s, A.partial, A.mblk, cfl,
                                               A.tau));
    else
      NS_LAUNCH("dt_final", hipLaunchKernelGGL(k_dt_final, dim3(1), dim3(1024), 0, s,
                                               A.partial, (int64_t)grid.x, cfl, A.tau));
  }
  if (G.byrow)
    NS_LAUNCH("lo", hipLaunchKernelGGL((k_lo_rows<DIM, LT>), grid, block, 0, s, G, A, gas));
  else
    NS_LAUNCH("lo", hipLaunchKernelGGL((k_lo<DIM, LT>), lgrid, block, 0, s, G, A, gas));
  if (limiter == 1) {
    NS_LAUNCH("combine", hipLaunchKernelGGL((k_combine_low<DIM, LT>), grid, block, 0, s,
                                            G, A));
  } else if (limiter == 2) {
    NS_LAUNCH("lim2", hipLaunchKernelGGL((k_lim2<DIM, 2, SEV, LT>), grid, block, 0, s, G, A,
                                         gas));
  } else {
    auto first = [&](auto keep) {
      constexpr bool KEEP = decltype(keep)::value;
      if (G.byrow)
        NS_LAUNCH("lim_first", hipLaunchKernelGGL((k_lim_first_rows<DIM, SEV, KEEP, LT>), grid,
                                                  block, 0, s, G, A, gas));
      else
        NS_LAUNCH("lim_first", hipLaunchKernelGGL((k_lim_first<DIM, SEV, KEEP, LT>), lgrid,
                                                  block, 0, s, G, A, gas));
    };
    auto two_passes = [&](auto keep) {
      constexpr bool KEEP = decltype(keep)::value;
      first(keep);
      if constexpr (DIM == 3) {
        const dim3 egrid(spec_slices(G.nsrow) + grid.x);
        NS_LAUNCH("lim_entries", hipLaunchKernelGGL((k_lim_entries<SEV, KEEP, LT>), egrid, block,
                                                    0, s, G, A, gas));
        NS_LAUNCH("fin", hipLaunchKernelGGL(k_fin_entries<LT>, egrid, block, 0, s, G, A));
      } else {
        const dim3 wide(kWide), rows(spec_groups(G) + lim_groups(G.N));
        if (G.byrow)
          NS_LAUNCH("lim_done", hipLaunchKernelGGL(k_lim_done_rows<LT>, grid, block, 0, s, G, A));
        else
          NS_LAUNCH("lim_done", hipLaunchKernelGGL(k_lim_done<LT>, grid, block, 0, s, G, A));
        NS_LAUNCH("lim_rows", hipLaunchKernelGGL((k_lim_rows<SEV, KEEP, LT>), rows, wide, 0, s,
                                                 G, A, gas));
        NS_LAUNCH("fin", hipLaunchKernelGGL(k_fin_rows<LT>, rows, wide, 0, s, G, A));
      }
    };
    if (passes != 1) {
      if (A.keep) two_passes(std::true_type{});
      else two_passes(std::false_type{});
    } else {
      // the work list holds a small fraction of the edges (~1.5% of them in the
      // 3D shock tube); up to 4M lanes cover a list without striding, and
      // blocks past its end exit at once
      const dim3 rgrid(std::min<unsigned>(grid.x, 16384u));
      NS_LAUNCH("lim1", hipLaunchKernelGGL((k_lim1<DIM, SEV, LT>), grid, block, 0, s, G, A,
                                           gas));
      NS_LAUNCH("root1", hipLaunchKernelGGL((k_root<DIM, SEV, LT>), rgrid, block, 0, s, G,
                                            A, gas));
      NS_LAUNCH("lim2", hipLaunchKernelGGL((k_lim2<DIM, 1, SEV, LT>), grid, block, 0, s, G,
                                           A, gas));
    }
  }
#undef NS_LAUNCH
}

template <int DIM, int SEV, typename LT>
void dt_impl(const Gas &gas, const DevGraphT<LT> &G, const StageArgsT<LT> &A, double cfl,
             hipStream_t s, void (*before)(void *, const char *),
             void (*after)(void *), void *prof) {
  const dim3 grid = grid_for(G.N), block(kBlock);
  const dim3 lgrid(grid.x + spec_blocks<DIM>(G));
  before(prof, "prim");
  hipLaunchKernelGGL(k_prim<DIM>, grid, block, 0, s, G.N, A.U, A.aux, gas,
                     (int *)nullptr);
  after(prof);
  before(prof, "visc_dt");
  if (G.byrow)
    hipLaunchKernelGGL((k_visc_rows<DIM, 2, SEV, LT>), grid, block, 0, s, G, A.U, A.aux, A.d,
                       A.alpha, gas);
  else
    hipLaunchKernelGGL((k_visc<DIM, 2, SEV, LT>), lgrid, block, 0, s, G, A.U, A.aux, A.d,
                       A.alpha, gas);
  after(prof);
  before(prof, "dt_partial");
  hipLaunchKernelGGL((k_dt_partial<DIM, LT>), grid, block, 0, s, G, A.d, A.partial);
  after(prof);
  before(prof, "dt_final");
  if (A.seg)
    hipLaunchKernelGGL(k_dt_final_members, dim3((unsigned)A.nmem), dim3(1024), 0, s,
                       A.partial, A.mblk, cfl, A.tau);
  else
    hipLaunchKernelGGL(k_dt_final, dim3(1), dim3(1024), 0, s, A.partial, (int64_t)grid.x,
                       cfl, A.tau);
  after(prof);
}

}  // namespace

template <typename LT>
void launch_dt_only(int dim, const Gas &gas, const DevGraphT<LT> &g,
                    const StageArgsT<LT> &a, double cfl, hipStream_t s,
                    void (*before)(void *, const char *), void (*after)(void *),
                    void *prof) {
  if (dim == 2) {
    if (gas.seven) dt_impl<2, 1, LT>(gas, g, a, cfl, s, before, after, prof);
    else dt_impl<2, 0, LT>(gas, g, a, cfl, s, before, after, prof);
  } else {
    if (gas.seven) dt_impl<3, 1, LT>(gas, g, a, cfl, s, before, after, prof);
    else dt_impl<3, 0, LT>(gas, g, a, cfl, s, before, after, prof);
  }
}

template <typename LT>
void launch_stage(int dim, const Gas &gas, const DevGraphT<LT> &g,
                  const StageArgsT<LT> &a, int indicator, int limiter, int passes,
                  bool auto_dt, double cfl, hipStream_t s,
                  void (*before)(void *, const char *), void (*after)(void *),
                  void *prof) {
  auto run = [&](auto impl) {
    impl(gas, g, a, indicator, limiter, passes, auto_dt, cfl, s, before, after, prof);
  };
  if (dim == 2) {
    if (gas.seven) run(stage_impl<2, 1, LT>);
    else run(stage_impl<2, 0, LT>);
  } else {
    if (gas.seven) run(stage_impl<3, 1, LT>);
    else run(stage_impl<3, 0, LT>);
  }
}

template void launch_stage<double>(int, const Gas &, const DevGraphT<double> &,
                                   const StageArgsT<double> &, int, int, int, bool,
                                   double, hipStream_t, void (*)(void *, const char *),
                                   void (*)(void *), void *);
template void launch_stage<float>(int, const Gas &, const DevGraphT<float> &,
                                  const StageArgsT<float> &, int, int, int, bool,
                                  double, hipStream_t, void (*)(void *, const char *),
                                  void (*)(void *), void *);
template void launch_dt_only<double>(int, const Gas &, const DevGraphT<double> &,
                                     const StageArgsT<double> &, double, hipStream_t,
                                     void (*)(void *, const char *), void (*)(void *),
                                     void *);
template void launch_dt_only<float>(int, const Gas &, const DevGraphT<float> &,
                                    const StageArgsT<float> &, double, hipStream_t,
                                    void (*)(void *, const char *), void (*)(void *),
                                    void *);

void launch_slip(int dim, int64_t N, int nslip, const int32_t *idx,
                 const double *nrm, double *U, hipStream_t s, int stride) {
  if (nslip <= 0) return;
  if (stride < 0) stride = nslip;
  const dim3 grid((unsigned)((nslip + kBlock - 1) / kBlock)), block(kBlock);
  if (dim == 2)
    hipLaunchKernelGGL(k_slip<2>, grid, block, 0, s, nslip, idx, nrm, stride, N, U);
  else
    hipLaunchKernelGGL(k_slip<3>, grid, block, 0, s, nslip, idx, nrm, stride, N, U);
}

void launch_set_scalar(double *p, double v, hipStream_t s, int n) {
  hipLaunchKernelGGL(k_set_scalar, dim3((unsigned)((n + 63) / 64)), dim3(64), 0, s, p, v, n);
}

void launch_add_scalar(double *acc, const double *v, hipStream_t s, int n) {
  hipLaunchKernelGGL(k_add_scalar, dim3((unsigned)((n + 63) / 64)), dim3(64), 0, s, acc, v,
                     n);
}

void launch_copy(const void *src, void *dst, int64_t n16, int word,
                 hipStream_t s) {
  if (word == 8)
    hipLaunchKernelGGL(k_copy8, grid_for(2 * n16), dim3(kBlock), 0, s,
                       static_cast<const double *>(src), static_cast<double *>(dst),
                       2 * n16);
  else
    hipLaunchKernelGGL(k_copy, grid_for(n16), dim3(kBlock), 0, s,
                       static_cast<const double2 *>(src),
                       static_cast<double2 *>(dst), n16);
}

void launch_nodes_from_cm(int nc, const double *src, int64_t ns, double *dst, int64_t N,
                          int64_t first, int64_t count, hipStream_t s) {
  if (count <= 0) return;
  if (nc == 4)
    hipLaunchKernelGGL(k_nodes_from_cm<4>, grid_for(count), dim3(kBlock), 0, s, src, ns, dst,
                       N, first, count);
  else
    hipLaunchKernelGGL(k_nodes_from_cm<5>, grid_for(count), dim3(kBlock), 0, s, src, ns, dst,
                       N, first, count);
}

void launch_nodes_to_cm(int nc, const double *src, int64_t N, int64_t first, int64_t count,
                        double *dst, int64_t ns, hipStream_t s) {
  if (count <= 0) return;
  if (nc == 4)
    hipLaunchKernelGGL(k_nodes_to_cm<4>, grid_for(count), dim3(kBlock), 0, s, src, N, first,
                       count, dst, ns);
  else
    hipLaunchKernelGGL(k_nodes_to_cm<5>, grid_for(count), dim3(kBlock), 0, s, src, N, first,
                       count, dst, ns);
}

void persist_plan(int dim, int64_t rows_tot, int64_t roots_tot, int64_t slips_tot,
                  int nmem, PersistPlan *pl) {
  int n = 0;
  auto add = [&](int ph, int st) {
    pl->phase[n] = (int8_t)ph;
    pl->stage[n] = (int8_t)st;
    ++n;
  };
  for (int st = 0; st < 3; ++st) {
    add(PP_PRIM, st);
    add(PP_VISC, st);
    if (st == 0) {  // the CFL time step of the step
      add(PP_DTP, st);
      add(PP_DTF, st);
    }
    add(PP_LO, st);
    add(PP_LIM1, st);
    add(PP_ROOT1, st);
    add(PP_LIM2, st);
    if (dim == 3) add(PP_LIM2B, st);
    add(PP_ROOT2, st);
    add(PP_FIN, st);
    add(PP_SLIP, st);
  }
  pl->nph = n;
  int16_t c[4] = {0, 0, 0, 0};
  int64_t off = 0;
  for (int p = 0; p <= n; ++p) {
    for (int k = 0; k < 4; ++k) pl->pre[p][k] = c[k];
    pl->off[p] = off;
    if (p == n) break;
    const int kind = persist_kind(pl->phase[p]);
    ++c[kind];
    off += kind == PK_ROW ? rows_tot : kind == PK_ROOT ? roots_tot
           : kind == PK_SLIP ? slips_tot : nmem;
  }
}

namespace {
template <typename F>
const void *persist_kernel(int dim, bool seven, F pick) {
  return dim == 2 ? (seven ? pick(std::integral_constant<int, 2>{}, std::integral_constant<int, 1>{})
                           : pick(std::integral_constant<int, 2>{}, std::integral_constant<int, 0>{}))
                  : (seven ? pick(std::integral_constant<int, 3>{}, std::integral_constant<int, 1>{})
                           : pick(std::integral_constant<int, 3>{}, std::integral_constant<int, 0>{}));
}
template <typename LT>
const void *persist_kernel_lt(int dim, bool seven) {
  return persist_kernel(dim, seven, [](auto d, auto sev) {
    return (const void *)k_persist<decltype(d)::value, decltype(sev)::value, LT>;
  });
}
}  // namespace

int persist_grid(int dim, bool seven, bool fp32) {
  const void *k = fp32 ? persist_kernel_lt<float>(dim, seven)
                       : persist_kernel_lt<double>(dim, seven);
  int dev = 0, cus = 0, per = 0;
  if (hipGetDevice(&dev) != hipSuccess) return 0;
  if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess)
    return 0;
  if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per, k, kBlock, 0) != hipSuccess) return 0;
  return std::max(per, 1) * cus;
}

template <typename LT>
void launch_persistent(int dim, const Gas &gas, const DevGraphT<LT> &g,
                       const PersistArgsT<LT> &p, int grid, hipStream_t s) {
  const dim3 gr((unsigned)grid), bl(kBlock);
  if (dim == 2) {
    if (gas.seven) hipLaunchKernelGGL((k_persist<2, 1, LT>), gr, bl, 0, s, g, p, gas);
    else hipLaunchKernelGGL((k_persist<2, 0, LT>), gr, bl, 0, s, g, p, gas);
  } else {
    if (gas.seven) hipLaunchKernelGGL((k_persist<3, 1, LT>), gr, bl, 0, s, g, p, gas);
    else hipLaunchKernelGGL((k_persist<3, 0, LT>), gr, bl, 0, s, g, p, gas);
  }
}
template void launch_persistent<double>(int, const Gas &, const DevGraphT<double> &,
                                        const PersistArgsT<double> &, int, hipStream_t);
template void launch_persistent<float>(int, const Gas &, const DevGraphT<float> &,
                                       const PersistArgsT<float> &, int, hipStream_t);

void launch_persist_reset(uint32_t *done, uint32_t *pcnt, uint32_t *ticket, int *stop,
                          int nmem, bool run_start, hipStream_t s) {
  hipLaunchKernelGGL(k_persist_reset, dim3((unsigned)((2 * nmem + 63) / 64)), dim3(64), 0, s,
                     done, pcnt, ticket, stop, nmem, run_start ? 1 : 0);
}

void launch_clear_flags(int *flags, hipStream_t s, int n) {
  hipLaunchKernelGGL(k_clear_flags, dim3((unsigned)((4 * n + 63) / 64)), dim3(64), 0, s,
                     flags, n);
}

template <typename LT>
int launch_stats(int dim, const DevGraphT<LT> &g, const double *U, const LT *lt1,
                 const LT *lt2, int mode, double *part, double *out, hipStream_t s) {
  const int nparts = (int)std::min<int64_t>((g.N + kBlock - 1) / kBlock, kStatsParts);
  if (dim == 2)
    hipLaunchKernelGGL((k_stats_partial<2, LT>), dim3(nparts), dim3(kBlock), 0, s, g, U, lt1,
                       lt2, mode, part);
  else
    hipLaunchKernelGGL((k_stats_partial<3, LT>), dim3(nparts), dim3(kBlock), 0, s, g, U, lt1,
                       lt2, mode, part);
  hipLaunchKernelGGL(k_stats_final, dim3(1), dim3(kBlock), 0, s, part, nparts, out);
  return nparts;
}
template int launch_stats<double>(int, const DevGraphT<double> &, const double *,
                                  const double *, const double *, int, double *, double *,
                                  hipStream_t);
template int launch_stats<float>(int, const DevGraphT<float> &, const double *, const float *,
                                 const float *, int, double *, double *, hipStream_t);

void launch_check_state(int dim, int64_t N, const double *U, int *flags,
                        hipStream_t s) {
  const dim3 grid = grid_for(N), block(kBlock);
  if (dim == 2)
    hipLaunchKernelGGL(k_check_state<2>, grid, block, 0, s, N, U, flags);
  else
    hipLaunchKernelGGL(k_check_state<3>, grid, block, 0, s, N, U, flags);
}

}  // namespace ns

// mg_kernels.hip -- geometric multigrid V-cycle in FP32 preconditioning the
// parabolic CG (the paper's viscous-dominated regime: a V-cycle in single
// precision with a Chebyshev-Jacobi smoother inside the double-precision CG).
//
// Smoother: Chebyshev iteration of degree deg for A x = b preconditioned by
// the diagonal D, on the interval [lmax/10, lmax] where lmax is the
// Gershgorin bound of D^-1 A (an upper bound of its spectrum, so the
// iteration cannot diverge); theta, delta the interval's centre and half
// width, sigma = theta/delta, rho_0 = 1/sigma, rho_k = 1/(2 sigma - rho_{k-1}):
//   d_0 = D^-1 r_0 / theta,  d_k = rho_k rho_{k-1} d_{k-1} + 2 rho_k/delta D^-1 r_k,
//   x_{k+1} = x_k + d_k,  r_k = b - A x_k.
// The same polynomial before and after the coarse correction and R = P^T
// make the V-cycle symmetric, as the preconditioned CG needs.  Rows of
// no-slip nodes (velocity) are kept at zero on every level.
#include "par_kernels.hpp"

#include <cmath>

#include "par_ops.hpp"

namespace ns {
namespace {
using namespace pops;

__device__ __forceinline__ int64_t mgid() {
  return (int64_t)blockIdx.x * kParBlock + threadIdx.x;
}
inline dim3 mgrid(int64_t n) { return dim3((unsigned)((n + kParBlock - 1) / kParBlock)); }

template <int DIM>
__device__ __forceinline__ bool wall_node(const ParGrid &G, const int64_t c[3]) {
  bool w = false;
#pragma unroll
  for (int d = 0; d < DIM; ++d)
    if (!G.per[d] && (c[d] == 0 || c[d] == G.n[d] - 1)) w = true;
  return w;
}

// coarse nodes (at most 2) and weights interpolating at fine index i of one
// direction: the fine node sits at i cc/cf coarse cells
__device__ __forceinline__ int interp1(int32_t i, int32_t nf, int32_t nc, int per,
                                       int32_t *I, float *w) {
  const int32_t cf = per ? nf : nf - 1, cc = per ? nc : nc - 1;
  const double xi = (double)i * (double)cc / (double)cf;
  const int32_t i0 = (int32_t)floor(xi);
  const double t = xi - (double)i0;
  if (!per && i0 >= cc) {
    I[0] = cc;
    w[0] = 1.0f;
    return 1;
  }
  I[0] = i0;
  w[0] = (float)(1.0 - t);
  if (!(t > 0.0)) return 1;
  I[1] = per && i0 + 1 == nc ? 0 : i0 + 1;
  w[1] = (float)t;
  return 2;
}

// Weight with which coarse index I enters the interpolation at fine index i:
// interp1's, with the same arithmetic.
__device__ __forceinline__ float weight1(int32_t i, int32_t I, int32_t nf, int32_t nc, int per) {
  int32_t J[2];
  float w[2];
  const int m = interp1(i, nf, nc, per, J, w);
  return J[0] == I ? w[0] : m > 1 && J[1] == I ? w[1] : 0.0f;
}

// Fine indices and weights with which coarse index I enters the interpolation,
// the transpose of interp1.  They lie in the open interval ((I-1) r, (I+1) r),
// r = cf / cc <= 2 fine cells to a coarse one: 4 at most (weight 0: none).
struct Fine4 {
  int32_t i[4];
  float w[4];
  __device__ __forceinline__ Fine4(int32_t I, int32_t nf, int32_t nc, int per) {
    const int32_t cf = per ? nf : nf - 1, cc = per ? nc : nc - 1;
    const int32_t j0 = (int32_t)floor((double)(I - 1) * (double)cf / (double)cc) + 1;
    const double end = (double)(I + 1) * (double)cf / (double)cc;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      int32_t j = j0 + q;
      const bool in = (double)j < end;
      if (per) j = j < 0 ? j + nf : j >= nf ? j - nf : j;
      const bool ok = in && j >= 0 && j < nf;
      j = ok ? j : 0;
      i[q] = j;
      w[q] = ok ? weight1(j, I, nf, nc, per) : 0.0f;
    }
  }
};

// acc = (R r)(c), get(j, rj) reading the components of r at fine node j
template <int DIM, int NC, class Get>
__device__ __forceinline__ void restrict_node(const ParGrid &Gf, const ParGrid &Gc,
                                              const int64_t c[3], const Get &get,
                                              float (&acc)[NC]) {
#pragma unroll
  for (int k = 0; k < NC; ++k) acc[k] = 0.0f;
  const Fine4 fx((int32_t)c[0], (int32_t)Gf.n[0], (int32_t)Gc.n[0], Gf.per[0]), fy((int32_t)c[1], (int32_t)Gf.n[1], (int32_t)Gc.n[1], Gf.per[1]);
  const int32_t n0 = (int32_t)Gf.n[0], n01 = n0 * (int32_t)Gf.n[1];
  auto plane = [&](int32_t z, float wz) {
#pragma unroll
    for (int b = 0; b < 4; ++b)
#pragma unroll
      for (int a = 0; a < 4; ++a) {
        const float ww = fx.w[a] * fy.w[b] * wz;
        float r[NC];
        get(fx.i[a] + n0 * fy.i[b] + z, r);
        if (ww != 0.0f) {
#pragma unroll
          for (int k = 0; k < NC; ++k) acc[k] += ww * r[k];
        }
      }
  };
  if constexpr (DIM == 2) {
    plane(0, 1.0f);
  } else {
    const Fine4 fz((int32_t)c[2], (int32_t)Gf.n[2], (int32_t)Gc.n[2], Gf.per[2]);
#pragma unroll
    for (int q = 0; q < 4; ++q)
      if (fz.w[q] != 0.0f) plane(n01 * fz.i[q], fz.w[q]);
  }
}

// b_c = R r_f; VEL: zero at no-slip coarse nodes.  All 16 (a plane's, in 3D)
// gathers are in flight at once and the weights stay in registers; as loops
// over the fine nodes found, with 64-bit remainders and the lists in scratch
// memory, it took 9.5 us (velocity) and 13.3 us (energy) per launch on the
// levels of 501 x 400, now 6.0 and 5.6 on the fine ones.
template <int DIM, int NC, bool VEL>
__global__ __launch_bounds__(kParBlock) void k_mg_restrict(ParGrid Gf, ParGrid Gc,
                                                           const float *__restrict__ rf,
                                                           float *__restrict__ bc,
                                                           const CGState *st) {
  if (st && st->done) return;
  const int64_t I = mgid();
  if (I >= Gc.N) return;
  int64_t c[3];
  decode(Gc, I, c);
  float acc[NC];
#pragma unroll
  for (int k = 0; k < NC; ++k) acc[k] = 0.0f;
  const int64_t N = Gf.N;
  if (!(VEL && wall_node<DIM>(Gc, c)))
    restrict_node<DIM, NC>(Gf, Gc, c, [=](int32_t j, float (&r)[NC]) {
#pragma unroll
      for (int k = 0; k < NC; ++k) r[k] = rf[k * N + j];
    }, acc);
#pragma unroll
  for (int k = 0; k < NC; ++k) bc[k * Gc.N + I] = acc[k];
}

// acc = (P x_c)(c), get(J, xJ) reading the components of x_c at coarse node J
template <int DIM, int NC, class Get>
__device__ __forceinline__ void prolong_node(const ParGrid &Gf, const ParGrid &Gc,
                                             const int64_t c[3], const Get &get,
                                             float (&acc)[NC]) {
  int32_t I[3][2];
  float w[3][2];
  bool two[3];
#pragma unroll
  for (int d = 0; d < DIM; ++d) {
    two[d] = interp1((int32_t)c[d], (int32_t)Gf.n[d], (int32_t)Gc.n[d], Gf.per[d], I[d], w[d]) > 1;
    if (!two[d]) I[d][1] = I[d][0];
  }
  const int32_t n0 = (int32_t)Gc.n[0], n01 = n0 * (int32_t)Gc.n[1];
#pragma unroll
  for (int k = 0; k < NC; ++k) acc[k] = 0.0f;
#pragma unroll
  for (int a2 = 0; a2 < (DIM == 3 ? 2 : 1); ++a2)
#pragma unroll
    for (int a1 = 0; a1 < 2; ++a1)
#pragma unroll
      for (int a0 = 0; a0 < 2; ++a0) {
        float x[NC];
        float ww = w[0][a0] * w[1][a1];
        int32_t J = I[0][a0] + n0 * I[1][a1];
        bool ok = (a0 == 0 || two[0]) && (a1 == 0 || two[1]);
        if constexpr (DIM == 3) {
          ww *= w[2][a2];
          J += n01 * I[2][a2];
          ok = ok && (a2 == 0 || two[2]);
        }
        get(J, x);
        if (ok) {
#pragma unroll
          for (int k = 0; k < NC; ++k) acc[k] += ww * x[k];
        }
      }
}

// x_f += P x_c; VEL: no-slip fine nodes untouched (they stay zero)
template <int DIM, int NC, bool VEL>
__global__ __launch_bounds__(kParBlock) void k_mg_prolong(ParGrid Gf, ParGrid Gc,
                                                          const float *__restrict__ xc,
                                                          float *__restrict__ xf,
                                                          const CGState *st) {
  if (st && st->done) return;
  const int64_t i = mgid();
  if (i >= Gf.N) return;
  int64_t c[3];
  decode(Gf, i, c);
  if (VEL && wall_node<DIM>(Gf, c)) return;
  float acc[NC];
  const int64_t N = Gc.N;
  prolong_node<DIM, NC>(Gf, Gc, c, [=](int32_t J, float (&x)[NC]) {
#pragma unroll
    for (int k = 0; k < NC; ++k) x[k] = xc[k * N + J];
  }, acc);
#pragma unroll
  for (int k = 0; k < NC; ++k) xf[k * Gf.N + i] += acc[k];
}

// diagonal and the Gershgorin ratio (rm + cdt sum_j |a_ij|) / (rm + cdt a_ii),
// row sums over the element entries of the node's cells (an upper bound of
// the assembled row's); block maxima into gpart
template <int DIM, int NC, bool VEL>
__global__ __launch_bounds__(kParBlock) void k_mg_diag(MGLevel L, float cdt) {
  constexpr int NL = 1 << DIM;
  const int64_t i = mgid();
  const int64_t N = L.G.N;
  float ratio = 0.0f;
  if (i < N) {
    int64_t c[3];
    decode(L.G, i, c);
    const bool fx = VEL && wall_node<DIM>(L.G, c);
    const float *E = L.tab + (NC > 1 ? 0 : TabOff<DIM>::heat);
    const float rm = L.rm[i];
#pragma unroll
    for (int k = 0; k < NC; ++k) {
      if (fx) {
        L.diag[k * N + i] = 1.0f;
        ratio = fmaxf(ratio, 1.0f);
        continue;
      }
      const float dk = rm + cdt * op_diag<DIM, NC, float>(L.G, E, c, k);
      float s = 0.0f;
      for (int a = 0; a < NL; ++a) {
        if (!cell_exists<DIM>(L.G, c, a)) continue;
        for (int b = 0; b < NL; ++b)
#pragma unroll
          for (int l = 0; l < NC; ++l) s += fabsf(E[((k * NC + l) * NL + a) * NL + b]);
      }
      L.diag[k * N + i] = dk;
      ratio = fmaxf(ratio, (rm + cdt * s) / dk);
    }
  }
  __shared__ float sh[kParBlock / 64];
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) ratio = fmaxf(ratio, __shfl_xor(ratio, off));
  if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = ratio;
  __syncthreads();
  if (threadIdx.x == 0) {
    for (int w = 1; w < kParBlock / 64; ++w) ratio = fmaxf(ratio, sh[w]);
    L.gpart[blockIdx.x] = ratio;
  }
}

__global__ __launch_bounds__(kParBlock) void k_mg_lmax(const float *__restrict__ gpart, int nb,
                                                       float *lmax) {
  float m = 0.0f;
  for (int j = threadIdx.x; j < nb; j += kParBlock) m = fmaxf(m, gpart[j]);
  __shared__ float sh[kParBlock / 64];
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) m = fmaxf(m, __shfl_xor(m, off));
  if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = m;
  __syncthreads();
  if (threadIdx.x == 0) {
    for (int w = 1; w < kParBlock / 64; ++w) m = fmaxf(m, sh[w]);
    *lmax = m;
  }
}

__global__ __launch_bounds__(kParBlock) void k_mg_narrow(int64_t n, const double *__restrict__ a,
                                                         float *__restrict__ b) {
  const int64_t t = mgid();
  if (t < n) b[t] = (float)a[t];
}

// level 0 right-hand side from the CG residual; VEL: zero at no-slip nodes
template <int DIM, int NC, bool VEL>
__global__ __launch_bounds__(kParBlock) void k_mg_from_residual(ParGrid G,
                                                                const double *__restrict__ r,
                                                                float *__restrict__ b,
                                                                const CGState *st) {
  if (st && st->done) return;
  const int64_t i = mgid();
  if (i >= G.N) return;
  int64_t c[3];
  decode(G, i, c);
  const bool fx = VEL && wall_node<DIM>(G, c);
#pragma unroll
  for (int k = 0; k < NC; ++k) b[k * G.N + i] = fx ? 0.0f : (float)r[k * G.N + i];
}

template <int NC>
__global__ __launch_bounds__(kParBlock) void k_mg_widen(int64_t N, const float *__restrict__ x,
                                                        double *__restrict__ z,
                                                        const CGState *st) {
  if (st && st->done) return;
  const int64_t t = mgid();
  if (t < NC * N) z[t] = (double)x[t];
}

// Chebyshev iteration k from xin to xout; FIRST: iterations 0 and 1 from zero.
// The iterate after iteration 0 is b / D / theta, which each lane forms at its
// neighbours itself: that saves a launch (2.6 us at 501 x 400) for the
// divisions, and the iterate and direction in between.
template <int DIM, int NC, bool VEL, bool FIRST>
__global__ __launch_bounds__(kParBlock) void k_mg_cheb(MGLevel L, float cdt, int k,
                                                       const float *__restrict__ xin,
                                                       float *__restrict__ xout,
                                                       const CGState *st) {
  if (st && st->done) return;
  const int64_t i = mgid();
  const int64_t N = L.G.N;
  if (i >= N) return;
  int64_t c[3];
  decode(L.G, i, c);
  if (VEL && wall_node<DIM>(L.G, c)) {
#pragma unroll
    for (int q = 0; q < NC; ++q) {
      xout[q * N + i] = 0.0f;
      L.d[q * N + i] = 0.0f;
    }
    return;
  }
  const float lmax = *L.lmax, lmin = 0.1f * lmax;
  const float theta = 0.5f * (lmax + lmin), delta = 0.5f * (lmax - lmin);
  const float sigma = theta / delta;
  float rho_prev = 1.0f / sigma, rho = rho_prev;
  for (int j = 1; j <= k; ++j) {
    rho_prev = rho;
    rho = 1.0f / (2.0f * sigma - rho_prev);
  }
  const float rm = L.rm[i];
  float acc[NC], xi[NC];
  if constexpr (FIRST) {
    const float *__restrict__ b = L.b, *__restrict__ dg = L.diag;
    // (b is 0 and D is 1 at the fixed nodes)
    const auto get = [=](int64_t j, float (&x)[NC]) {
#pragma unroll
      for (int q = 0; q < NC; ++q) x[q] = b[q * N + j] / dg[q * N + j] / theta;
    };
    op_near<DIM, NC, float>(Near<DIM>(L.G, c), stencil_of<DIM, NC>(L.tab),
                            element_of<DIM, NC>(L.tab), get, acc);
    get(i, xi);
  } else {
    op_apply<DIM, NC, float>(L.G, L.tab, xin, c, acc);
#pragma unroll
    for (int q = 0; q < NC; ++q) xi[q] = xin[q * N + i];
  }
#pragma unroll
  for (int q = 0; q < NC; ++q) {
    const float r = L.b[q * N + i] - (rm * xi[q] + cdt * acc[q]);
    const float zr = r / L.diag[q * N + i];
    const float dp = FIRST ? xi[q] : k == 0 ? 0.0f : L.d[q * N + i];
    const float d = k == 0 ? zr / theta : rho * rho_prev * dp + 2.0f * rho / delta * zr;
    L.d[q * N + i] = d;
    xout[q * N + i] = xi[q] + d;
  }
}

// res = b - A x (VEL: zero at no-slip nodes)
template <int DIM, int NC, bool VEL>
__global__ __launch_bounds__(kParBlock) void k_mg_residual(MGLevel L, float cdt,
                                                           const float *__restrict__ x,
                                                           float *__restrict__ res,
                                                           const CGState *st) {
  if (st && st->done) return;
  const int64_t i = mgid();
  const int64_t N = L.G.N;
  if (i >= N) return;
  int64_t c[3];
  decode(L.G, i, c);
  if (VEL && wall_node<DIM>(L.G, c)) {
#pragma unroll
    for (int q = 0; q < NC; ++q) res[q * N + i] = 0.0f;
    return;
  }
  float acc[NC];
  op_apply<DIM, NC, float>(L.G, L.tab, x, c, acc);
  const float rm = L.rm[i];
#pragma unroll
  for (int q = 0; q < NC; ++q) res[q * N + i] = L.b[q * N + i] - (rm * x[q * N + i] + cdt * acc[q]);
}

// ---------------------------------------------------------------------------
// The coarse levels of a V-cycle in one workgroup.  Below a few thousand nodes
// a level's kernels cost their launch (3 - 4 us each, 30 of the 55 of a
// V-cycle at 501 x 400), while one CU runs an iteration in 0.3 - 1 us from
// LDS: the levels from the first with at most kTailNodes nodes on (and whose
// iterates fit kTailWords) go through one kernel.  The line lies where one
// CU's iteration costs what a launch does: 4096 nodes of 9 neighbours, 1024
// of 27 (a parabolic step with no such levels / up to 1024 / 2048 / 4096 nodes:
// 12^3 2.53 / 2.11 / 2.34 / 2.41 ms, 24^3 3.50 / 3.05 / 3.05 / 3.63, 48^3 4.99 /
// 4.51 / 4.49 / 5.17, 101 x 67 x 83 9.15 / 8.60 / 8.92 / 9.05).  A lane owns up
// to NPT nodes of a level: its right-hand side, direction and diagonal stay in
// registers while it smooths, the two buffers of the iterate are in LDS; b of the
// levels below goes through global memory between lanes of the same number only
// (coarse node I is restricted and smoothed by lane I mod kTailThreads).  501 x 400
// (levels of 3264, 858 and 238 nodes): 53 us (velocity) and 46 us (energy) for
// 30 launches before, about 120 and 180 us; most of it the arithmetic of the
// largest level, 3 us per iteration on one CU's SIMDs.
constexpr int kTailThreads = 1024, kTailWords = 24576;
template <int DIM> constexpr int kTailPer = DIM == 2 ? 4 : 1;  // nodes of a lane
template <int DIM> constexpr int kTailNodes = kTailPer<DIM> * kTailThreads;
constexpr int kTailLevels = 16;
struct MGTail {
  MGLevel lv[kTailLevels];
  int off[kTailLevels];  // first word of a level's buffers
  int n;
};

// A value that all lanes hold, in a scalar register.
__device__ __forceinline__ float scalar(float x) {
  return __int_as_float(__builtin_amdgcn_readfirstlane(__float_as_int(x)));
}

// (no element matrix: velocity rows of wall nodes are fixed)
struct NoTable {
  __device__ __forceinline__ float operator[](int) const { return 0.0f; }
};

template <int DIM, int NC, bool VEL> struct TailLevel {
  static constexpr int NPT = kTailPer<DIM>;
  using O = TabOff<DIM>;
  // 2D: the tables stay in scalar registers (read per node and iteration, the
  // wait for them was most of the time)
  static constexpr bool KEPT = DIM == 2;
  static constexpr int NS = KEPT ? O::S * NC * NC : 1, NE = KEPT && !VEL ? O::L * O::L : 1;
  const MGLevel &L;
  float *sh;  // two buffers of NC * N words
  const int N, tid;
  float st[NS], E[NE];
  __device__ __forceinline__ TailLevel(const MGTail &T, int l, float *words)
      : L(T.lv[l]), sh(words + T.off[l]), N((int)T.lv[l].G.N), tid((int)threadIdx.x) {}
  __device__ __forceinline__ void tables() {
    if constexpr (KEPT) {
#pragma unroll
      for (int t = 0; t < NS; ++t)
        st[t] = scalar(stencil_of<DIM, NC>(L.tab)[t]);
      if constexpr (!VEL) {
#pragma unroll
        for (int t = 0; t < NE; ++t) E[t] = scalar(element_of<DIM, NC>(L.tab)[t]);
      }
    }
  }
  // the operator at a node (VEL: an interior one)
  __device__ __forceinline__ void apply(const Near<DIM> &nr, int h, float (&acc)[NC]) const {
    if constexpr (!KEPT)
      op_near<DIM, NC, float>(nr, stencil_of<DIM, NC>(L.tab), element_of<DIM, NC>(L.tab),
                              reader(h), acc);
    else if constexpr (VEL)
      op_near<DIM, NC, float>(nr, st, NoTable(), reader(h), acc);
    else
      op_near<DIM, NC, float>(nr, st, E, reader(h), acc);
  }
  __device__ __forceinline__ float *buf(int h) const { return sh + h * NC * N; }
  __device__ __forceinline__ auto reader(int h) const {
    const float *x = buf(h);
    const int n = N;
    return [=](int32_t j, float (&xj)[NC]) {
#pragma unroll
      for (int l = 0; l < NC; ++l) xj[l] = x[l * n + j];
    };
  }

  // deg Chebyshev iterations from buffer h (zero if zs); returns the buffer
  // that holds the result, not yet synchronised
  __device__ __forceinline__ int smooth(int h, int deg, bool zs, float cdt) const {
    float b[NPT][NC], rdg[NPT][NC], d[NPT][NC], rm[NPT];
    Near<DIM> nr[NPT];
#pragma unroll
    for (int m = 0; m < NPT; ++m) {
      const int i = tid + m * kTailThreads;
      if (i >= N) continue;
      rm[m] = L.rm[i];
      int64_t c[3];
      decode(L.G, i, c);
      nr[m] = Near<DIM>(L.G, c);
#pragma unroll
      for (int q = 0; q < NC; ++q) {
        b[m][q] = L.b[q * N + i];
        rdg[m][q] = 1.0f / L.diag[q * N + i];
        d[m][q] = 0.0f;
      }
    }
    const float lmax = *L.lmax, lmin = 0.1f * lmax;
    const float theta = 0.5f * (lmax + lmin), delta = 0.5f * (lmax - lmin);
    const float sigma = theta / delta;
    float rho_prev = 1.0f / sigma, rho = rho_prev;
    for (int k = 0; k < deg; ++k, h ^= 1) {
      if (k > 0) {
        rho_prev = rho;
        rho = 1.0f / (2.0f * sigma - rho_prev);
      }
      const bool zero = zs && k == 0;
      if (!zero) __syncthreads();
      const float *xin = buf(h);
      float *xout = buf(h ^ 1);
#pragma unroll
      for (int m = 0; m < NPT; ++m) {
        const int i = tid + m * kTailThreads;
        if (i >= N) continue;
        if (VEL && !nr[m].interior()) {
#pragma unroll
          for (int q = 0; q < NC; ++q) xout[q * N + i] = 0.0f;
          continue;
        }
        float r[NC];
        if (zero) {
#pragma unroll
          for (int q = 0; q < NC; ++q) r[q] = b[m][q];
        } else {
          float acc[NC];
          apply(nr[m], h, acc);
#pragma unroll
          for (int q = 0; q < NC; ++q)
            r[q] = b[m][q] - (rm[m] * xin[q * N + i] + cdt * acc[q]);
        }
#pragma unroll
        for (int q = 0; q < NC; ++q) {
          const float zr = r[q] * rdg[m][q];
          d[m][q] = k == 0 ? zr / theta : rho * rho_prev * d[m][q] + 2.0f * rho / delta * zr;
          xout[q * N + i] = (zero ? 0.0f : xin[q * N + i]) + d[m][q];
        }
      }
    }
    return h;
  }

  // b - A x of buffer h into the other
  __device__ __forceinline__ void residual(int h, float cdt) const {
    const float *x = buf(h);
    float *res = buf(h ^ 1);
    for (int i = tid; i < N; i += kTailThreads) {
      int64_t c[3];
      decode(L.G, i, c);
      const Near<DIM> nr(L.G, c);
      const bool fx = VEL && !nr.interior();
      float acc[NC];
      apply(nr, h, acc);
      const float rm = L.rm[i];
#pragma unroll
      for (int q = 0; q < NC; ++q)
        res[q * N + i] = fx ? 0.0f : L.b[q * N + i] - (rm * x[q * N + i] + cdt * acc[q]);
    }
  }
};

// From b of its first level to that level's x.
template <int DIM, int NC, bool VEL>
__global__ __launch_bounds__(kTailThreads) void k_mg_tail(MGTail T, float cdt, int deg, int cdeg,
                                                          const CGState *st) {
  using TL = TailLevel<DIM, NC, VEL>;
  __shared__ float words[kTailWords];
  if (st && st->done) return;
  const int tid = (int)threadIdx.x;
  uint32_t at = 0;  // bit l: buffer that holds level l's iterate
  for (int l = 0; l + 1 < T.n; ++l) {
    TL F(T, l, words);
    F.tables();
    const int h = F.smooth(0, deg, true, cdt);
    at |= (uint32_t)h << l;
    __syncthreads();
    F.residual(h, cdt);
    __syncthreads();
    const MGLevel &C = T.lv[l + 1];
    for (int I = tid; I < (int)C.G.N; I += kTailThreads) {
      int64_t c[3];
      decode(C.G, I, c);
      float acc[NC];
      if (VEL && wall_node<DIM>(C.G, c)) {
#pragma unroll
        for (int q = 0; q < NC; ++q) acc[q] = 0.0f;
      } else {
        restrict_node<DIM, NC>(F.L.G, C.G, c, F.reader(h ^ 1), acc);
      }
#pragma unroll
      for (int q = 0; q < NC; ++q) C.b[q * C.G.N + I] = acc[q];
    }
  }
  {
    TL C(T, T.n - 1, words);
    C.tables();
    at |= (uint32_t)C.smooth(0, cdeg, true, cdt) << (T.n - 1);
  }
  for (int l = T.n - 2; l >= 0; --l) {
    TL F(T, l, words), C(T, l + 1, words);
    F.tables();
    const int h = (at >> l) & 1;
    __syncthreads();
    const auto coarse = C.reader((at >> (l + 1)) & 1);
    float *x = F.buf(h);
    for (int i = tid; i < F.N; i += kTailThreads) {
      int64_t c[3];
      decode(F.L.G, i, c);
      if (VEL && wall_node<DIM>(F.L.G, c)) continue;
      float acc[NC];
      prolong_node<DIM, NC>(F.L.G, C.L.G, c, coarse, acc);
#pragma unroll
      for (int q = 0; q < NC; ++q) x[q * F.N + i] += acc[q];
    }
    at = (at & ~(1u << l)) | (uint32_t)F.smooth(h, deg, false, cdt) << l;
  }
  const TL F(T, 0, words);
  const float *x = F.buf(at & 1);
  for (int i = tid; i < F.N; i += kTailThreads)
#pragma unroll
    for (int q = 0; q < NC; ++q) F.L.x[q * F.N + i] = x[q * F.N + i];
}

// First level of the tail (nlev: none), filling T.
template <int DIM, int NC> int tail_levels(const MGLevel *lv, int nlev, MGTail *T) {
  int first = nlev;
  int64_t words = 0;
  while (first > 0 && nlev - first < kTailLevels && lv[first - 1].G.N <= kTailNodes<DIM> &&
         words + 2 * NC * lv[first - 1].G.N <= kTailWords)
    words += 2 * NC * lv[--first].G.N;
  T->n = nlev - first;
  int off = 0;
  for (int l = 0; l < T->n; ++l) {
    T->lv[l] = lv[first + l];
    T->off[l] = off;
    off += 2 * NC * (int)lv[first + l].G.N;
  }
  return first;
}

template <int DIM, int NC, bool VEL>
void setup_t(MGLevel *lv, int nlev, const double *rm, double cdt, hipStream_t s) {
  hipLaunchKernelGGL(k_mg_narrow, mgrid(lv[0].G.N), dim3(kParBlock), 0, s, lv[0].G.N, rm,
                     lv[0].rm);
  for (int l = 1; l < nlev; ++l)
    hipLaunchKernelGGL((k_mg_restrict<DIM, 1, false>), mgrid(lv[l].G.N), dim3(kParBlock), 0, s,
                       lv[l - 1].G, lv[l].G, (const float *)lv[l - 1].rm, lv[l].rm,
                       (const CGState *)nullptr);
  for (int l = 0; l < nlev; ++l) {
    const dim3 g = mgrid(lv[l].G.N);
    hipLaunchKernelGGL((k_mg_diag<DIM, NC, VEL>), g, dim3(kParBlock), 0, s, lv[l], (float)cdt);
    hipLaunchKernelGGL(k_mg_lmax, dim3(1), dim3(kParBlock), 0, s, (const float *)lv[l].gpart,
                       (int)g.x, lv[l].lmax);
  }
}

// smooth `deg` >= 2 times on level l starting from *cur (zero if zs); the
// iterate alternates between the level's x and y; returns the result
template <int DIM, int NC, bool VEL>
float *smooth(const MGLevel &L, float *cur, int deg, int zs, float cdt, const CGState *st,
              hipStream_t s) {
  const dim3 g = mgrid(L.G.N);
  for (int k = zs ? 1 : 0; k < deg; ++k) {
    float *out = cur == L.x ? L.y : L.x;
    if (zs && k == 1)
      hipLaunchKernelGGL((k_mg_cheb<DIM, NC, VEL, true>), g, dim3(kParBlock), 0, s, L, cdt, k,
                         (const float *)nullptr, out, st);
    else
      hipLaunchKernelGGL((k_mg_cheb<DIM, NC, VEL, false>), g, dim3(kParBlock), 0, s, L, cdt, k,
                         (const float *)cur, out, st);
    cur = out;
  }
  return cur;
}

template <int DIM, int NC, bool VEL>
float *vcycle_level(const MGLevel *lv, int l, int nlev, const MGTail &T, float cdt,
                    const CGState *st, int deg, int coarse_deg, hipStream_t s) {
  const MGLevel &L = lv[l];
  if (l == nlev - T.n) {
    hipLaunchKernelGGL((k_mg_tail<DIM, NC, VEL>), dim3(1), dim3(kTailThreads), 0, s, T, cdt, deg,
                       coarse_deg, st);
    return L.x;
  }
  if (l == nlev - 1) return smooth<DIM, NC, VEL>(L, L.x, coarse_deg, 1, cdt, st, s);
  float *cur = smooth<DIM, NC, VEL>(L, L.x, deg, 1, cdt, st, s);
  float *res = cur == L.x ? L.y : L.x;
  const dim3 g = mgrid(L.G.N), gc = mgrid(lv[l + 1].G.N);
  hipLaunchKernelGGL((k_mg_residual<DIM, NC, VEL>), g, dim3(kParBlock), 0, s, L, cdt,
                     (const float *)cur, res, st);
  hipLaunchKernelGGL((k_mg_restrict<DIM, NC, VEL>), gc, dim3(kParBlock), 0, s, L.G, lv[l + 1].G,
                     (const float *)res, lv[l + 1].b, st);
  const float *xc =
      vcycle_level<DIM, NC, VEL>(lv, l + 1, nlev, T, cdt, st, deg, coarse_deg, s);
  hipLaunchKernelGGL((k_mg_prolong<DIM, NC, VEL>), g, dim3(kParBlock), 0, s, L.G, lv[l + 1].G, xc,
                     cur, st);
  return smooth<DIM, NC, VEL>(L, cur, deg, 0, cdt, st, s);
}

template <int DIM, int NC, bool VEL>
void vcycle_t(const MGLevel *lv, int nlev, const double *r, double *z, double cdt,
              const CGState *st, int deg, int coarse_deg, hipStream_t s) {
  const dim3 g = mgrid(lv[0].G.N);
  MGTail T;
  (void)tail_levels<DIM, NC>(lv, nlev, &T);
  hipLaunchKernelGGL((k_mg_from_residual<DIM, NC, VEL>), g, dim3(kParBlock), 0, s, lv[0].G, r,
                     lv[0].b, st);
  const float *x =
      vcycle_level<DIM, NC, VEL>(lv, 0, nlev, T, (float)cdt, st, deg, coarse_deg, s);
  hipLaunchKernelGGL(k_mg_widen<NC>, mgrid(NC * lv[0].G.N), dim3(kParBlock), 0, s, lv[0].G.N, x,
                     z, st);
}

}  // namespace

void mg_setup(int dim, int ncomp, MGLevel *lv, int nlev, const double *rm, double cdt,
              hipStream_t s) {
  if (dim == 2) {
    if (ncomp == 2) setup_t<2, 2, true>(lv, nlev, rm, cdt, s);
    else setup_t<2, 1, false>(lv, nlev, rm, cdt, s);
  } else {
    if (ncomp == 3) setup_t<3, 3, true>(lv, nlev, rm, cdt, s);
    else setup_t<3, 1, false>(lv, nlev, rm, cdt, s);
  }
}

void mg_vcycle(int dim, int ncomp, const MGLevel *lv, int nlev, const double *r, double *z,
               double cdt, const CGState *st, int deg, int coarse_deg, hipStream_t s) {
  if (dim == 2) {
    if (ncomp == 2) vcycle_t<2, 2, true>(lv, nlev, r, z, cdt, st, deg, coarse_deg, s);
    else vcycle_t<2, 1, false>(lv, nlev, r, z, cdt, st, deg, coarse_deg, s);
  } else {
    if (ncomp == 3) vcycle_t<3, 3, true>(lv, nlev, r, z, cdt, st, deg, coarse_deg, s);
    else vcycle_t<3, 1, false>(lv, nlev, r, z, cdt, st, deg, coarse_deg, s);
  }
}

}  // namespace ns

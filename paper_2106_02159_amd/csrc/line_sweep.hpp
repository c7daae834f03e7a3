// line_sweep.hpp -- neighbour access of the row sweeps along stencil lines.
//
// A row whose 3^d neighbours all exist without crossing a periodic seam (an
// interior row) has its neighbours at the same row offsets as every other
// interior row of its mesh: (dx, dy, dz) -> dx + n0 (dy + n1 dz).  The rows of
// a wavefront are consecutive, so the neighbours of one line (dy, dz) are the
// 64 consecutive nodes of that line and one node beyond either end.  A sweep
// loads a line once, coalesced, from a wave-uniform base address, plus the
// two end nodes in lanes 0 and 63, and takes the dx = -1 and dx = +1
// neighbours from the lanes beside it (DPP wavefront shifts).  Against one
// gather per slot this is a third of the load instructions and L1 accesses,
// three memory round trips per row in 2D instead of nine, no address
// arithmetic per lane, and the coefficients m_ij, c_ij, |c_ij| and n_ij of
// an entry come from the mesh's table in scalar registers.
//
// All other rows (a few in a thousand on a large 2D mesh, 3% at 192^3) are
// listed once per solver; workgroups at the front of the same launch run them
// through the general per-slot path, one lane per row and line.  (Meshes a few
// nodes thick, mostly such rows, take every row by itself: many_listed.)
//
// Per launch, gather per slot -> along lines (FP64): graph viscosity 0.81 ->
// 0.54 ms at 4096^2, 1.06 -> 0.79 ms at 192^3; low-order sweep 1.09 -> 0.73
// and 1.37 -> 0.95 ms.  VALU instructions per row fall from 1176 to 790 and
// from 1059 to 770 in 2D.
#pragma once

#include <cstdint>
#include <type_traits>

#include <hip/hip_runtime.h>

#include "box_nbr.hpp"
#include "node_layout.hpp"

namespace ns {

// Lane l receives x of lane l - 1 (lane 0: `end` of lane 0), and of lane
// l + 1 (lane 63: `end` of lane 63).  Every lane of the wave must be active.
template <int CTRL>
__device__ __forceinline__ double wave_shift(double end, double x) {
  const int2 e = __builtin_bit_cast(int2, end), s = __builtin_bit_cast(int2, x);
  int2 r;
  r.x = __builtin_amdgcn_update_dpp(e.x, s.x, CTRL, 0xf, 0xf, false);
  r.y = __builtin_amdgcn_update_dpp(e.y, s.y, CTRL, 0xf, 0xf, false);
  return __builtin_bit_cast(double, r);
}
__device__ __forceinline__ double from_left(double end, double x) {
  return wave_shift<0x138>(end, x);  // wave_shr:1
}
__device__ __forceinline__ double from_right(double end, double x) {
  return wave_shift<0x130>(end, x);  // wave_shl:1
}

constexpr int kLineRows = 256;  // rows of a workgroup

// The rows b + c (the lane's own place on the line) and, in lanes 0 and 63,
// b + h (the node beyond the wave's end).  b is uniform over the workgroup;
// rows beyond the array are replaced by the nearest one in it (their values
// are never used by an interior row).
struct Line {
  int64_t b;
  uint32_t c, h;
};

__device__ __forceinline__ Line make_line(int64_t r0, int64_t delta, int64_t N,
                                          uint32_t tid) {
  Line L;
  L.b = r0 + delta - 1;
  const int64_t last = N - 1;
  if (L.b > last || L.b < -(int64_t)(kLineRows + 1)) L.b = 0;
  const int lo = L.b < 0 ? (int)-L.b : 0;
  const int hi = (int)(last - L.b < (int64_t)(kLineRows + 1) ? last - L.b
                                                              : (int64_t)(kLineRows + 1));
  const int c = (int)tid + 1, h = (tid & 63) == 0 ? c - 1 : c + 1;
  L.c = (uint32_t)min(max(c, lo), hi);
  L.h = (uint32_t)min(max(h, lo), hi);
  return L;
}

// Called where a line starts: the loads of later lines depend on nothing
// before them, and without it the compiler issues them all first and keeps
// them live.  Emits no instruction.
__device__ __forceinline__ void line_fence(uint32_t &tid) {
  asm volatile("" : "+v"(tid) : : "memory");
  __builtin_amdgcn_sched_barrier(0);
}
// A row's running sums at the end of a line: they are only stored at the end
// and only by interior rows, and without it the compiler moves all of the
// row's arithmetic there, with every line's data live.
template <typename... T>
__device__ __forceinline__ void line_keep(T &...v) {
  (([](T &x) { asm volatile("" : "+v"(x)); })(v), ...);
}

// A wave-uniform global address as such: the offset of the lane is then added
// by the load itself (scalar base, 32-bit lane offset).
__device__ __forceinline__ uint32_t from_left(uint32_t end, uint32_t x) {
  return __builtin_amdgcn_update_dpp((int)end, (int)x, 0x138, 0xf, 0xf, false);
}
__device__ __forceinline__ uint32_t from_right(uint32_t end, uint32_t x) {
  return __builtin_amdgcn_update_dpp((int)end, (int)x, 0x130, 0xf, 0xf, false);
}

template <typename T>
using vec2 = T __attribute__((ext_vector_type(2)));
template <typename T>
using global_ptr = __attribute__((address_space(1))) T *;
template <typename T>
__device__ __forceinline__ global_ptr<T> uniform_ptr(T *p) {
  const uint64_t a = reinterpret_cast<uint64_t>(p);
  const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)a);
  const uint32_t hi = __builtin_amdgcn_readfirstlane((uint32_t)(a >> 32));
  return (global_ptr<T>)((uint64_t)hi << 32 | lo);
}
// Entry e of an array at a uniform address.
template <typename T>
__device__ __forceinline__ global_ptr<T> lane_at(T *base, uint32_t e) {
  using B = std::conditional_t<std::is_const_v<T>, const char, char>;
  return (global_ptr<T>)((global_ptr<B>)uniform_ptr(base) + e * (uint32_t)sizeof(T));
}
template <typename T>
__device__ __forceinline__ std::remove_const_t<T> line_ld(T *p, int64_t b, uint32_t off) {
  return *lane_at(p + b, off);
}

// f(integral_constant<int, I>) for I = 0 .. N-1.
template <int I, int N, typename F>
__device__ __forceinline__ void static_for(F &&f) {
  if constexpr (I < N) {
    f(std::integral_constant<int, I>{});
    static_for<I + 1, N>(f);
  }
}

}  // namespace ns

// row_lists.hpp -- lists of the rows that a 2D limiter stage has to work on.
//
// Limited rows come in fronts and patches: a fixed share of the mesh for each
// workgroup leaves the work to the few whose share holds them, and whatever
// stride or skew spreads one line length over the workgroups lines up with
// another (4096 x 4150 with a front along y, slices of 64 rows dealt out with a
// skew of 37: 28 times the mean on the fullest workgroup, k_lim_rows 0.36 ms per
// stage, k_fin_rows 0.13; by these lists 0.055 and 0.026).  So the blocks of
// 256 rows append their marked rows to lists, and the waves of the next
// kernels take equal parts of the lists.
//
// One counter would serialise the appends (15 ns each): there are up to 64
// lists, 32 bytes between their counters.  A list holds the rows of at most
// ceil(blocks / lists) blocks: each group of `lists` blocks maps onto the lists
// one to one, rotated by a hash of the group's number so that a mesh line that
// is a multiple of the group does not bring a front to a few of the lists.
#pragma once

#include <cstdint>

#include <hip/hip_runtime.h>

namespace ns {

constexpr uint32_t kListRows = 256;  // rows of a block
constexpr uint32_t kMaxLists = 64;
constexpr uint32_t kListStep = 8;    // words from one list's counter to the next

struct RowLists {
  uint32_t lists;  // power of two
  uint32_t room;   // rows of a list
  __host__ __device__ explicit RowLists(uint32_t blocks) : lists(1) {
    while (lists < kMaxLists && 2 * lists <= blocks) lists *= 2;
    room = (blocks + lists - 1) / lists * kListRows;
  }
  __host__ __device__ uint32_t list_of(uint32_t block) const {
    return (block + ((block / lists) * 0x9e3779b1u >> 26)) & (lists - 1);
  }
};

// The parts of `each` rows that the workgroups take in turn: part p is the rows
// from p / lists * each on of list p % lists.  In this order (and not list by
// list) rows that are near in the mesh are worked on at about the same time and
// find each other's data in the caches; 64 rows to 8 waves of 8, fewer where
// they would not reach all workgroups.  All rows of 2048 x 2048 limited,
// k_lim_rows and k_fin_rows per stage: 0.66 and 0.31 ms, list by list 0.71
// and 0.34.
__host__ __device__ inline uint32_t part_rows(uint32_t longest, uint32_t lists, uint32_t groups) {
  const uint32_t per = longest * lists / groups;  // (longest * lists <= 2 N + 2^14)
  return per >= 56 ? 64 : (per + 8) / 8 * 8;
}

}  // namespace ns

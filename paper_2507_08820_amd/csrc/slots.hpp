// slots.hpp -- where the kernels around the step find a node's populations in the
// AA layout of kernels.hpp: at an even step count f_i(x) sits in slot A[i][x],
// at an odd one in A[26 - i][x - c_i].
#pragma once
#include <cstdint>
#include <hip/hip_runtime.h>

#include "d3q27.hpp"
#include "kernels.hpp"
#include "storage.hpp"

namespace rflbm {

struct NodeXYZ {
  uint32_t x, y, z;
};

__device__ __forceinline__ NodeXYZ coords(uint64_t n, uint32_t nx, uint32_t ny) {
  NodeXYZ c;
  c.x = static_cast<uint32_t>(n % nx);
  const uint64_t r = n / nx;
  c.y = static_cast<uint32_t>(r % ny);
  c.z = static_cast<uint32_t>(r / ny);
  return c;
}

// Element index of slot A[plane][(x, y, z)] in the x-row blocked layout, its
// row blocks in By x Bz bricks (kernels.hpp; By = Bz = 1: plain layout).
__device__ __forceinline__ uint64_t element_index(int plane, uint32_t x, uint32_t y, uint32_t z,
                                                  const GatherArgs& g) {
  const uint64_t yo = (y >> g.by_log) * g.ybrick_pitch + (y & ((1u << g.by_log) - 1u)) * g.row_pitch;
  const uint64_t zo = (z >> g.bz_log) * g.plane_pitch + (z & ((1u << g.bz_log) - 1u)) * g.zin_pitch;
  return zo + yo + static_cast<uint64_t>(plane) * g.pop_pitch + x;
}

// Element index of the slot holding f_i(x) at the given parity.
__device__ __forceinline__ uint64_t slot_index(int i, NodeXYZ p, const GatherArgs& g) {
  if (!g.odd) return element_index(i, p.x, p.y, p.z, g);
  const int cx = i % 3 - 1, cy = (i / 3) % 3 - 1, cz = i / 9 - 1;
  return element_index(kQ - 1 - i, wrap_add(p.x, -cx, g.nx), wrap_add(p.y, -cy, g.ny),
                       wrap_add(p.z, -cz, g.nz), g);
}

// Node n < 2^32 -> (x, y, z) with two magic divisions.
__device__ __forceinline__ NodeXYZ coords32(uint32_t n, const GatherArgs& g) {
  NodeXYZ c;
  const uint32_t r = fast_div(n, g.div_x);
  c.x = n - r * g.nx;
  c.z = fast_div(r, g.div_y);
  c.y = r - c.z * g.ny;
  return c;
}

// Element indices of the 27 slots of one node: the row blocks (and x positions)
// they lie in are found once, a slot is then one of them plus its population row.
template <bool ODD>
struct Slots {
  uint64_t row[9];  // row block of (y - c_y, z - c_z), at c_y + 1 + 3 (c_z + 1); even: row[4] only
  uint32_t xs[3];   // x - c_x, at c_x + 1
  uint32_t pitch;
  __device__ __forceinline__ Slots(NodeXYZ p, const GatherArgs& g) : pitch(static_cast<uint32_t>(g.pop_pitch)) {
    if constexpr (ODD) {
#pragma unroll
      for (int c = -1; c <= 1; ++c) xs[c + 1] = wrap_add(p.x, -c, g.nx);
#pragma unroll
      for (int q = 0; q < 9; ++q)
        row[q] = element_index(0, 0, wrap_add(p.y, 1 - q % 3, g.ny), wrap_add(p.z, 1 - q / 3, g.nz), g);
    } else {
      row[4] = element_index(0, p.x, p.y, p.z, g);
    }
  }
  __device__ __forceinline__ uint64_t operator()(int i) const {
    if constexpr (ODD) return row[i / 3] + (xs[i % 3] + static_cast<uint32_t>(kQ - 1 - i) * pitch);
    else return row[4] + static_cast<uint32_t>(i) * pitch;
  }
};

}  // namespace rflbm

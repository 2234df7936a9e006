// sk.hpp -- structure-factor kernels (sk.hip) as api.cpp launches them.
#pragma once
#include <cstdint>
#include <hip/hip_runtime.h>

#include "kernels.hpp"
#include "policy.hpp"

namespace rflbm {

// Blocks (and partial sums) per field of the last pass, at most: with ten fields
// one round of the two such blocks a CU holds.
constexpr uint32_t kSkBlocks = 51;

// The pass along x: pairs of rows per block, values of one field's spectrum.
struct SkRows {
  uint32_t pairs;
  uint64_t pitch;
  FastDiv div_lines;  // division by the complex lines of a block
  FastDiv div_hx;     // division by nx / 2 + 1
};

// A pass along y or z: lines in tiles of 2^log_tx neighbouring columns.
struct SkTiles {
  uint32_t hx;      // nx / 2 + 1
  uint32_t lines;   // lines of one field
  uint32_t log_tx;
  uint32_t threads;
  uint64_t pitch;
  FastDiv div_hx, div_tx;
};

// Blocks per field of the last pass: partial holds 10 sk_blocks nshells doubles.
uint32_t sk_blocks(uint32_t nx, uint32_t ny, uint32_t nz);
// Adds |F|^2 / N of the ten fields of the state g to shell_sum[10][nshells] and
// writes the new sums to host_sum (pinned host memory) too.
// twiddle: exp(-2 pi i t / n) for the sides nx, ny, nz one after another; spec:
// 10 (nx / 2 + 1) ny nz complex values of scratch.
hipError_t launch_sk(int storage, const GatherArgs& g, const float2* twiddle, uint32_t nshells, float2* spec,
                     double* partial, double* shell_sum, double* host_sum, hipStream_t s);
// Adds the wavevectors per shell to shell_count.
hipError_t launch_sk_count(uint32_t nx, uint32_t ny, uint32_t nz, uint32_t nshells, unsigned long long* shell_count,
                           hipStream_t s);
// Copies n 8-byte words, in stream order.
hipError_t launch_sk_copy(const void* src, uint32_t n, void* dst, hipStream_t s);
// Shell sums of one field's stored spectrum.
hipError_t launch_sk_bin(const void* spec, uint32_t nx, uint32_t ny, uint32_t nz, uint32_t nshells,
                         double* shell_sum, hipStream_t s);

}  // namespace rflbm

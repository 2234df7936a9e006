// policy.hpp -- which kernel a call takes, as rules on sizes alone: plain host code
// without HIP, so that the rules can be checked where there is no GPU.
#pragma once
#include <cstdint>

namespace rflbm {

constexpr uint32_t kFftMaxLength = 1024;  // of the transforms in LDS (fft.hpp)

// Grid of 256-thread blocks, one thread a node: block x + y kNodeGridX covers the nodes
// from 256 times that.  A launch takes fewer than 2^32 threads along an axis, so the
// largest boxes (below 2^32 nodes) go over two.
constexpr uint64_t kNodeGridX = 1ull << 23;
struct NodeGrid {
  uint32_t x, y;
};
inline NodeGrid node_grid(uint64_t nodes) {
  const uint64_t blocks = (nodes + 255) / 256, x = blocks < kNodeGridX ? blocks : kNodeGridX;
  return NodeGrid{static_cast<uint32_t>(x), static_cast<uint32_t>((blocks + x - 1) / x)};
}

constexpr uint32_t kLineBytes = 128;           // cache line
constexpr uint64_t kCacheBytes = 256ull << 20;  // memory-side cache of an MI355X (Infinity Cache)

// True when a read of all populations goes past the caches: more than the
// memory-side cache holds, and each cache line read by one wave only, so even step
// counts (odd ones read rows shifted by one) and rows of whole lines.  Moment fields:
// 192^3 FP32 0.197 -> 0.173 ms, 256^3 FP16 0.295 -> 0.253; not so 130 x 101 x 97 BF16
// (in the cache) 0.023 -> 0.030, 255 x 256 x 200 FP16 0.227 -> 0.286, 288 x 256 x 256
// FP16 (4.5 lines a row) 0.322 -> 0.339, 200^3 FP16 0.138 -> 0.164.
inline bool read_streams(uint64_t row_bytes, uint64_t pop_bytes, bool odd) {
  return !odd && pop_bytes > kCacheBytes && row_bytes % kLineBytes == 0;
}

// One box as the choice of its step kernel sees it.
struct StepBox {
  uint32_t nx;
  uint32_t value_bytes;  // of a stored population
  bool noise;
  bool row_blocks;       // blocks that follow the rows, not tiles alone
  bool in_4gib;          // populations within 4 GiB
  bool in_turn;          // stepped in turn with others
  uint64_t turn_bytes;   // populations stepped in turn with these, and these
};

// kTiles: step_kernel, kFlat: step_flat_kernel, kRows: step_row_kernel, kWaves: step_wave_kernel.
enum class StepRoute { kTiles, kFlat, kRows, kWaves };

// Memory, not arithmetic, holds these steps: FP32, and 16 bits without noise.
inline bool memory_bound(const StepBox& b) { return b.value_bytes == 4 || !b.noise; }

// Non-temporal accesses of the steps that have them: even ones in waves, both
// parities in rows, even ones in flat blocks.
//
// Rows of whole waves, beyond 320 MiB (us a step with / without, FP32: 216 MiB
// (128^3) 81 / 65, 270 MiB 103 / 84, 338 MiB 126 / 123, 506 MiB 184 / 197, 1.7 GiB
// (256^3) 599 / 653; FP16 without noise 324 MiB 134 / 137, 864 MiB 303 / 328); beyond
// 1024 nodes, where odd steps are not in whole rows, beyond 256 MiB (1280 x 64 x 32
// FP32, 270 MiB, 86 / 96, 1920 x 64 x 22 90 / 98, 1280 x 64 x 64 FP16 without noise 90 / 103),
// and so boxes stepped in turn (10 x 64^3 FP32, 270 MiB, 62 / 64 a round of steps) and 16
// bits with noise (256 x 256 x 80 FP16, 270 MiB, 104 / 111, 192 x 192 x 140
// 102 / 110, 256 x 256 x 72, 243 MiB, 91 / 85).
// Memory-bound steps also from 6 to 18.5 MiB, FP32 with noise from 4 to 24, where the
// eight L2s (32 MiB) hold the default policy's dirty lines of one step when the next
// wants them on other XCDs (FP32 with noise 64 x 64 x 20 5.8 / 6.1, 64 x 64 x 32 6.3 / 7.1, 64
// x 64 x 48 7.5 / 8.5; 64 x 64 x 6, 3 MiB, 4.8 / 4.7, 64 x 64 x 60, 25 MiB, 9.3 / 9.1, 64^3 10.3 / 9.5;
// without noise 64 x 64 x 28 5.7 / 5.8, 320 x 21 x 25, 17.3 MiB, statistics every fifth step,
// 9.5 / 11.1, 64 x 64 x 44, 19 MiB, 7.1 / 6.9; FP16 without noise
// 64^3 7.5 / 7.6, 1280 x 16 x 16 8.2 / 8.8, 4096 x 8 x 8 7.3 / 8.4; 4096 x 16 x 16, 54 MiB, 21 / 17).
// Flat blocks: FP32 rows of whole or half lines beyond 256 MiB (160 x 160 x 100, 264 MiB,
// 85 / 95, 96 x 256 x 256 235 / 265, 416 x 200 x 200 647 / 688, 16 x 700 x 700 321 / 338);
// other rows share their lines with neighbours (300 x 200 x 100 318 / 255, 96^2 x
// 300 FP16 201 / 196).
inline bool step_streams(const StepBox& b) {
  if (b.nx % 64 != 0) return b.value_bytes == 4 && b.nx % 16 == 0 && b.turn_bytes > kCacheBytes;
  if (memory_bound(b) && b.turn_bytes >= (b.noise ? 4ull : 6ull) << 20 && 2 * b.turn_bytes <= (b.noise ? 48ull : 37ull) << 20)
    return true;
  const bool whole_rows = memory_bound(b) && b.nx <= 1024;
  return b.turn_bytes > (whole_rows && !b.in_turn ? 320ull << 20 : kCacheBytes);
}

// Blocks a CU is held to by steps in waves and in rows, 0: as many as fit (32 waves).
// Memory-bound steps that stream from memory reach 1 to 4 % more of its rate with
// about half the waves, hence fewer accesses in flight (us a step with 32 / fewer).
// FP32, 20 blocks of a wave and rows of 14 to 20 waves: BGK 384 x 207 x 247 769 / 742,
// 512 x 256 x 128 618 / 597 and with statistics 635 / 601, 128 x 256 x 512 629 / 608, 1024 x 128 x
// 128 635 / 623; two blocks at least (one: 1024 x 128 x 128 644, 768 x 200 x 150 864 / 902).
// Rows of an odd number of waves gain up to seven waves, without noise up to nine
// (448 x 200 x 200 with statistics 683 / 660, 320 x 256 x 200 620 / 611, but with noise 617 / 637;
// 960 x 60 x 61 139.2 / 139.7, 1088 x 64 x 64 159 / 161).
// 16 bits without noise, 16 blocks of a wave and rows of up to three waves at 18 to 20
// (BF16 BGK 192 x 256 x 300 276 / 269 in waves, 276 / 272 in rows, 320 x 226 x 191 265 / 258;
// rows of 16 waves 128 x 299 x 397 with statistics 288 / 298, of 384 nodes 372 / 461).
// In the cache and with noise in 16 bits fewer waves lose (64^3 8.4 / 9.1, 192^3 FP16 294 /
// 309, 320 x 256 x 200 FP16 330 / 347).
struct StepBlocks {
  uint32_t waves, rows;
};
inline StepBlocks step_blocks(const StepBox& b) {
  if (!memory_bound(b) || b.nx % 64 != 0 || b.turn_bytes <= kCacheBytes || !step_streams(b)) return {0, 0};
  const uint32_t waves = b.nx / 64;
  if (b.value_bytes != 4) return {16, waves <= 3 ? 20 / waves : 0};
  if (waves % 2 == 1 && waves >= 5 && (b.noise ? waves != 7 : waves > 9)) return {0, 0};
  return {20, waves < 8 ? 16 / waves : 2};
}

// The kernel of one step.
//
// Rows that do not fill waves, within 4 GiB: flat blocks, which leave no lane idle
// (figures at step_flat_kernel).  Beyond 256 MiB, where the odd step streams from memory,
// tiles keep what they lose few lanes on: rows of 33 to 63 nodes (FP32 63 x 300 x
// 140 flat 114, tiles 98, 56 x 200 x 300 141 / 124, 48 x 300 x 300 187 / 161; from 45 in 16
// bits, 63 x 300 x 280 FP16 143 / 118, 58 x 400 x 400 245 / 208, but 40 x 400 x 400 164 / 171),
// and FP32 rows of whole or half lines that fill 15 of 16 lanes of their tiles of 256
// (736 x 100 x 96 265 streamed, tiles 258, 2016 x 48 x 48 172 / 167, 1008 x 80 x 80 261 /
// 251; but 464 x 120 x 120 275 / 274, 352 x 256 x 128 439 / 456).
//
// Rows of whole waves: memory-bound steps in whole rows up to 1024 nodes (odd ones,
// and even ones with statistics: one partial a row, not one a wave), else in waves.
// Odd steps of longer rows in tiles of 256 where these fit: FP32 rows of a multiple
// of 128 (1280 x 64 x 64 191 / 202 us a step in waves, 1920 x 64 x 96 461 / 474, 1152 x 96
// x 96 412 / 424; 1088 x 64 x 64 163 / 159), 16 bits of a multiple of 256 when they
// stream (2048 x 64 x 64 FP16 158 / 160, 1792 x 48 x 64 98 / 101; in the cache 1088 x 64
// x 64 57 / 55).
// 16 bits with noise, bound by arithmetic, in waves of both parities: there the
// lane moves and barriers of the whole-row odd step cost more than aligned accesses
// save (512^3 3.8 / 3.2 ms), and waves leave no lane idle (us a step in waves / tiles of
// 128 or 256: 192^3 FP16 140 / 177, 320 x 96 x 96 FP16 55 / 83, 192 x 128 x 128 BF16
// 57 / 75, 128^3 FP16 40.4 / 43.8), except where tiles of 256 fit the rows and the box
// streams from memory (256^3 341 / 336, 512^3 2773 / 2713).
inline StepRoute step_route(const StepBox& b, bool odd, bool stats) {
  if (!b.row_blocks) return StepRoute::kTiles;
  const bool f32 = b.value_bytes == 4;
  if (b.nx % 64 != 0) {
    if (!b.in_4gib) return StepRoute::kTiles;
    if (b.turn_bytes > kCacheBytes) {
      if (b.nx >= (f32 ? 33u : 45u) && b.nx <= 63) return StepRoute::kTiles;
      const uint32_t lanes = (b.nx + 255) / 256 * 256;
      if (f32 && b.nx % 16 == 0 && b.nx >= 256 && 16 * b.nx >= 15 * lanes) return StepRoute::kTiles;
    }
    return StepRoute::kFlat;
  }
  if (memory_bound(b)) {
    if ((odd || stats) && b.nx <= 1024) return StepRoute::kRows;
    if (stats) return StepRoute::kTiles;
    return odd && (f32 ? b.nx % 128 == 0 : b.nx % 256 == 0 && step_streams(b)) ? StepRoute::kTiles : StepRoute::kWaves;
  }
  if (stats || (b.nx % 256 == 0 && step_streams(b))) return StepRoute::kTiles;
  return StepRoute::kWaves;
}

// Batches.  pop_bytes: populations of all replicas; rows: the greatest common
// divisor of their population-row lengths in bytes.
//
// Streaming batches are larger than what the memory-side cache keeps from step to
// step.  Whole-line rows lose the cache at its size (3 x 96^3 FP32, 273 MiB: 113 us a
// step, streamed 97; 90 of 32^3, 304 MiB: 105, 103), others a little beyond it
// (26 x 48^3, 296 MiB: 122, streamed 126; 60 x 48^3, 683 MiB: 324, 300).
inline bool batch_streams(uint64_t pop_bytes, uint64_t rows) {
  return pop_bytes > (rows % kLineBytes == 0 ? kCacheBytes : 320ull << 20);
}

// Non-temporal accesses of an even step of a streaming batch.  They fetch or write
// a line once for every population row that shares it, which pays in FP32 with at
// least half lines and in 16 bits with whole ones (us a step, non-temporal /
// default: 64 of 32^3..96^3 FP32 959 / 1013, 60 x 48^3 FP32 300 / 324, 4 x 128^3
// FP16 187 / 195; but 12 x 100^3 FP32 793 / 618, 20 of 130 x 50 x 70 FP32 596 / 458,
// 64 of 32^3..96^3 FP16 568 / 551, 32 x 96^3 FP16 781 / 748).  A sampled step also
// leaves its partials in the caches for the kernel that adds them: whole sectors are
// enough (64 of 32^3..96^3 FP16 with statistics every other step 602 / 621, 16 of
// them 236 / 246; 12 x 100^3 FP16 528 / 473), or replicas so large that this kernel,
// a block a replica, weighs more than the step (200^3 FP16 859 / 947, 180^3 606 / 695,
// 144^3 FP32 264 / 292).
inline bool batch_even_nt(uint64_t pop_bytes, uint64_t rows, bool f32, bool stats, uint64_t largest_nodes) {
  if (stats && pop_bytes > kCacheBytes && largest_nodes > (rows % 32 == 0 ? 1u << 21 : 1u << 22)) return true;
  if (!batch_streams(pop_bytes, rows)) return false;
  return rows % (f32 ? kLineBytes / 2 : kLineBytes) == 0 || (stats && rows % 32 == 0);
}

// One range of tiles per XCD instead of tiles dealt in turn: neighbouring tiles then
// meet in its L2, 8 x 20^3 FP32 7.6 -> 5.5 us a step, 24 of 8^3..32^3 FP16 7.4 -> 6.5,
// 8 x 64^3 FP32 69 -> 67.  Streaming batches lose by it (4 x 128^3 FP32 340 -> 350, 64 of
// 32^3..96^3 FP32 959 -> 989, 40 x 64^3 FP16 232 -> 237, 12 x 100^3 FP32 618 -> 647), but for
// FP32 beyond 2 GiB at one block a tile (64 of 32^3..96^3 835 -> 829, 32 x 96^3 1098
// -> 1073; 30 of 32^3..96^3, 1.3 GiB, 475 -> 487).
inline bool batch_in_ranges(uint64_t pop_bytes, uint64_t rows, bool f32, bool block_a_tile) {
  return !batch_streams(pop_bytes, rows) || (f32 && block_a_tile && pop_bytes > 2ull << 30);
}

// Largest prime factor of n >= 2.
inline uint32_t largest_prime(uint32_t n) {
  uint32_t p = 1;
  for (uint32_t d = 2; n > 1; ++d)
    for (; n % d == 0; n /= d) p = d;
  return p;
}

// True when the transforms in LDS take the box, else hipFFT.  A factor above 7
// costs them r operations a value where hipFFT has radices up to 17 and goes
// another way beyond.  ms of a snapshot, in LDS / hipFFT:
//  - one long prime side costs most along z and least along x, where hipFFT is
//    slowest: 32 x 32 x 1021 2.1 / 0.56, 45 x 45 x 331 0.72 / 0.60, 26 x 199 x 199
//    0.94 / 0.78, 32 x 1021 x 32 1.25 / 0.61, 1021 x 32 x 32 1.86 / 0.99; but 72 x 72 x
//    199 0.62 / 0.64, 32 x 509 x 32 0.42 / 0.45, 509 x 45 x 45 0.93 / 1.2; in a
//    few x-rows the launches weigh more: 8 x 8 x 509 0.19 / 0.30, 1021 x 2 x 2 0.86 / 0.39;
//  - beyond 2^20 nodes no prime above 64 (137 x 149 x 151 3.6 / 2.6);
//  - even nx, factors 11, 13, 17: 238^3 2.0 / 2.6, 242^3 2.6 / 2.6, 260^3 4.3 / 2.9,
//    286^3 7.9 / 3.8, 286 x 256 x 256 3.0 / 2.3, 256 x 256 x 286 3.1 / 3.0; such a side
//    along y alone is no loss (256 x 286 x 256 2.4 / 3.0), nor is odd nx (255^3
//    2.4 / 5.4, 363^3 12.0 / 15.7);
//  - even nx, factors of 19 to 61: 222^3 3.0 / 3.5, 212^3 3.2 / 3.3, 236^3 4.3 / 4.0,
//    244^3 4.7 / 4.1, 344^3 14.4 / 13.0, 366^3 22 / 15; but 290^3 8.3 / 8.6, 348^3
//    11.7 / 13.4, 406^3 16 / 20.
inline bool sk_fits(uint32_t nx, uint32_t ny, uint32_t nz) {
  if (nx > kFftMaxLength || ny > kFftMaxLength || nz > kFftMaxLength) return false;
  const auto factor = [](uint32_t n) {  // 0: radices of the transforms in LDS alone
    const uint32_t p = largest_prime(n);
    return p > 7 ? p : 0u;
  };
  const uint32_t rx = factor(nx), ry = factor(ny), rz = factor(nz);
  const uint32_t sum = rx + ry + rz, most = rx > ry ? (rx > rz ? rx : rz) : (ry > rz ? ry : rz);
  const uint64_t nodes = static_cast<uint64_t>(nx) * ny * nz;
  if (sum == 0) return true;
  if (nodes <= (1u << 17)) return rx <= 400 && rz <= 600;
  if (rx / 560.0 + ry / 510.0 + rz / 250.0 > 1.0) return false;
  if (nodes <= (1u << 20)) return true;
  if (most > 64) return false;
  if (nx % 2 != 0) return true;
  if (most <= 17) return nodes <= 27ull << 19 || sum == ry;
  return sum <= 100 || nodes * sum <= 1800000000ull;
}

}  // namespace rflbm

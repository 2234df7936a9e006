// sk.hip -- static structure factor (arXiv:2507.08820, Sec. III: spectra of a
// normalised FFT averaged over wavevectors of equal modulus).
//
// F(n) = sum_x dm(x) exp(-2 pi i n.x / L) of each of the ten moment fields; for
// every n != 0, |F(n)|^2 / N is added to shell round(|n|) with n_a taken in
// (-L_a/2, L_a/2].  Only kx = 0..nx/2 is formed; the other half of the spectrum
// is the complex conjugate (real input), so every column except kx = 0 and kx =
// nx/2 (nx even) counts twice.
//
// Sides up to 1024 (and see below): three passes over the data.
//   sk_rows_kernel: moments of whole x-rows and their transforms along x, two
//     rows of a field to one complex line, so no field is stored in real space;
//   sk_columns_kernel: along y, in place;
//   sk_shells_kernel: along z, and straight from LDS into shell sums, so the
//     transforms are not written again.
// Reads and writes are of 8 bytes x 16 neighbouring columns; a block's lines fill
// 32 KiB of LDS.  The floor is memory (256^3 FP32: 0.38 + 0.21 + 0.10 ms at copy
// rate); measured 0.51 + 0.31 + 0.30 ms, the last two held by the LDS passes and
// their index arithmetic.  A snapshot, against moment fields, one hipFFT
// transform and one binning kernel per field (43 launches): 256^3 FP32 1.06 / 2.62
// ms, 128^3 FP16 0.12 / 0.78, 64^3 0.032 / 0.21, 16^3 0.021 / 0.11, 200 x 320 x
// 180 BF16 0.78 / 2.16.
// The other way stays for sides beyond 1024 (LDS), and where the sums of prime
// factors above 7 cost more than hipFFT's transforms (sk_fits, policy.hpp).
#include <hip/hip_runtime.h>

#include <cstdint>
#include <type_traits>

#include "fft.hpp"
#include "sk.hpp"
#include "slots.hpp"

namespace rflbm {

namespace {

constexpr int kHalf = 5;  // fields transformed together: half of the ten

// Shell round(sqrt(k2)), exact: s with s (s - 1) < k2 <= s (s + 1).
__device__ __forceinline__ uint32_t shell_of(uint32_t k2) {
  uint32_t s = static_cast<uint32_t>(sqrtf(static_cast<float>(k2)) + 0.5f);
  if (s * (s + 1) < k2) ++s;
  else if (s * s - s >= k2 && s > 0) --s;
  return s;
}

// Square of the signed wavenumber of index k on a side of n.
__device__ __forceinline__ uint32_t wave2(uint32_t k, uint32_t n) {
  const uint32_t a = k <= n / 2 ? k : n - k;
  return a * a;
}

// Blocks of `pairs` pairs of x-rows (plane order).  A thread forms the moments of
// its node in both rows of a pair; each field of the pair is one complex line,
// five fields at a time, and its transform c splits as a = (c(k) + c*(-k)) / 2,
// b = (c(k) - c*(-k)) / 2i into those of the two rows.  Two rows of one field and
// not two fields: the smaller part of a line takes the rounding of the larger,
// and fields may differ by any factor (a flow without noise).  Two fields to a line,
// one of them 1e-4 (1e-6) of the other, had shell sums 2e-4 (2e-2) off, against
// 2e-7 for rows (64^3), and a field that overflowed took its partner with it.
template <int S, bool ODD, int KIND>
__global__ void __launch_bounds__(1024) sk_rows_kernel(const GatherArgs g, const FftPlan p, const SkRows r,
                                                       float2* __restrict__ spec) {
  using C = Codec<S>;
  using T = typename C::T;
  extern __shared__ float2 sh[];
  const uint32_t nx = g.nx, lines = kHalf * r.pairs;
  float2* const lds = sh;
  float2* const tw = sh + static_cast<size_t>(nx) * lines;
  const uint32_t tid = threadIdx.x;
  for (uint32_t t = tid; t < nx; t += blockDim.x) tw[t] = p.twiddle[t];
  const uint32_t total = g.ny * g.nz, row0 = blockIdx.x * 2 * r.pairs;
  const uint32_t pairs = min(r.pairs, (total - row0 + 1) >> 1);
  const uint32_t q = fast_div(tid, g.div_x), x = tid - q * nx;
  float f[2][2 * kHalf];  // the node's fields in the two rows (no second row: 0)
  if (q < pairs) {
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const uint32_t row = row0 + 2 * q + h;
      if (row < total) {
        NodeXYZ c;
        c.x = x;
        c.z = fast_div(row, g.div_y);
        c.y = row - c.z * g.ny;
        const Slots<ODD> slot(c, g);
        const T* pop = static_cast<const T*>(g.pop);
        float v[kQ];
#pragma unroll
        for (int i = 0; i < kQ; ++i) v[i] = C::decode(pop[slot(i)], g.sigma[speed_class(i)]);
        forward27(v);
        // rho - rho0 instead of rho: the mean does not enter n != 0
#pragma unroll
        for (int k = 0; k < 2 * kHalf; ++k) f[h][k] = v[mode_slot(k)];
      } else {
#pragma unroll
        for (int k = 0; k < 2 * kHalf; ++k) f[h][k] = 0.0f;
      }
    }
  }
  const uint32_t hx = nx / 2 + 1;
#pragma unroll
  for (int half = 0; half < 2; ++half) {
    if (q < pairs) {
#pragma unroll
      for (int k = 0; k < kHalf; ++k)
        lds[x * lines + q * kHalf + k] = make_float2(f[0][half * kHalf + k], f[1][half * kHalf + k]);
    }
    fft_lines<KIND>(lds, tw, lines, r.div_lines, p, tid, blockDim.x);
    for (uint32_t e = tid; e < pairs * kHalf * hx; e += blockDim.x) {
      const uint32_t l = fast_div(e, r.div_hx), k = e - l * hx;
      const uint32_t pair = l / kHalf, field = half * kHalf + l - pair * kHalf;
      const float2 c = lds[k * lines + l], d = lds[(k == 0 ? 0 : nx - k) * lines + l];
      const uint32_t row = row0 + 2 * pair;
      float2* const at = spec + field * r.pitch + static_cast<uint64_t>(row) * hx + k;
      at[0] = make_float2(0.5f * (c.x + d.x), 0.5f * (c.y - d.y));
      if (row + 1 < total) at[hx] = make_float2(0.5f * (c.y + d.y), 0.5f * (d.x - c.x));
    }
    if (half == 0) __syncthreads();  // the lines are written again
  }
}

// Along y, in place: block (tile, field); line l = kz hx + kx.  Each XCD (blocks
// b mod 8) takes one range of tiles, so that neighbouring tiles meet in its L2
// on the cache lines between them (256^3: 0.39 -> 0.36 ms for the ten fields).
template <int KIND>
__global__ void __launch_bounds__(512, KIND == kFftPow2 ? 8 : 1)
    sk_columns_kernel(const FftPlan p, const SkTiles c, float2* __restrict__ spec) {
  extern __shared__ float2 sh[];
  const uint32_t tx = 1u << c.log_tx, tid = threadIdx.x, n = p.n;
  float2* const lds = sh;
  float2* const tw = sh + (static_cast<size_t>(n) << c.log_tx);
  for (uint32_t t = tid; t < n; t += blockDim.x) tw[t] = p.twiddle[t];
  const uint32_t col = tid & (tx - 1u), pos0 = tid >> c.log_tx, dpos = blockDim.x >> c.log_tx;
  const uint32_t tile = (blockIdx.x & 7u) * (gridDim.x >> 3) + (blockIdx.x >> 3);
  const uint32_t l = (tile << c.log_tx) + col, kz = fast_div(l, c.div_hx);
  float2* const at = spec + blockIdx.y * c.pitch + (static_cast<uint64_t>(kz) * n * c.hx + (l - kz * c.hx));
  float2 v[kFftPerThread];
#pragma unroll
  for (int i = 0; i < kFftPerThread; ++i) {
    const uint32_t pos = pos0 + i * dpos;
    if (pos < n && l < c.lines) v[i] = at[static_cast<uint64_t>(pos) * c.hx];
  }
#pragma unroll
  for (int i = 0; i < kFftPerThread; ++i) {
    const uint32_t pos = pos0 + i * dpos;
    if (pos < n) lds[pos * tx + col] = v[i];
  }
  fft_lines<KIND>(lds, tw, tx, c.div_tx, p, tid, blockDim.x);
#pragma unroll
  for (int i = 0; i < kFftPerThread; ++i) {
    const uint32_t pos = pos0 + i * dpos;
    if (pos < n && l < c.lines) at[static_cast<uint64_t>(pos) * c.hx] = lds[pos * tx + col];
  }
}

// Along z and into shell sums: blocks (b, field) walk the tiles b, b + gridDim.x,
// ... of lines l = ky hx + kx.  +kz and -kz lie in one shell and are added
// before the LDS atomic; neighbouring columns, often of one shell too, go to
// different copies of the sums.  partial[(field gridDim.x + b) nshells + shell].
template <int KIND>
__global__ void __launch_bounds__(512) sk_shells_kernel(const FftPlan p, const SkTiles c, uint32_t nx, uint32_t ny,
                                                        uint32_t nshells, uint32_t log_copies, double inv_n,
                                                        const float2* __restrict__ spec,
                                                        double* __restrict__ partial) {
  extern __shared__ float2 sh[];
  const uint32_t tx = 1u << c.log_tx, tid = threadIdx.x, n = p.n, copies = 1u << log_copies;
  float2* const lds = sh;
  float2* const tw = sh + (static_cast<size_t>(n) << c.log_tx);
  double* const hist = reinterpret_cast<double*>(tw + n);
  for (uint32_t t = tid; t < n; t += blockDim.x) tw[t] = p.twiddle[t];
  for (uint32_t t = tid; t < nshells * copies; t += blockDim.x) hist[t] = 0.0;
  const uint32_t col = tid & (tx - 1u), pos0 = tid >> c.log_tx, dpos = blockDim.x >> c.log_tx;
  const uint32_t tiles = (c.lines + tx - 1) >> c.log_tx;
  float2 v[kFftPerThread];
  const auto load = [&](uint32_t l) {
    const float2* const at = spec + blockIdx.y * c.pitch + l;
#pragma unroll
    for (int i = 0; i < kFftPerThread; ++i) {
      const uint32_t pos = pos0 + i * dpos;
      if (pos < n && l < c.lines) v[i] = at[static_cast<uint64_t>(pos) * c.lines];
    }
  };
  load((blockIdx.x << c.log_tx) + col);
  for (uint32_t tile = blockIdx.x; tile < tiles; tile += gridDim.x) {
    const uint32_t l = (tile << c.log_tx) + col;
    const bool in = l < c.lines;
#pragma unroll
    for (int i = 0; i < kFftPerThread; ++i) {
      const uint32_t pos = pos0 + i * dpos;
      if (pos < n) lds[pos * tx + col] = v[i];
    }
    load(((tile + gridDim.x) << c.log_tx) + col);  // while this tile is transformed
    fft_lines<KIND>(lds, tw, tx, c.div_tx, p, tid, blockDim.x);
    if (in) {
      const uint32_t ky = fast_div(l, c.div_hx), kx = l - ky * c.hx;
      const uint32_t kxy2 = kx * kx + wave2(ky, ny);
      const double mult = (kx == 0 || 2 * kx == nx ? 1.0 : 2.0) * inv_n;
      double* const mine = hist + (col & (copies - 1u)) * nshells;
      for (uint32_t pos = pos0; pos <= n / 2; pos += dpos) {
        const uint32_t k2 = kxy2 + pos * pos;
        const float2 a = lds[pos * tx + col];
        double w = static_cast<double>(a.x) * a.x + static_cast<double>(a.y) * a.y;
        if (pos != 0 && 2 * pos != n) {
          const float2 b = lds[(n - pos) * tx + col];
          w += static_cast<double>(b.x) * b.x + static_cast<double>(b.y) * b.y;
        }
        if (k2 != 0) unsafeAtomicAdd(&mine[shell_of(k2)], w * mult);
      }
    }
    __syncthreads();
  }
  __syncthreads();
  double* const out = partial + (static_cast<size_t>(blockIdx.y) * gridDim.x + blockIdx.x) * nshells;
  for (uint32_t s = tid; s < nshells; s += blockDim.x) {
    double sum = 0.0;
    for (uint32_t k = 0; k < copies; ++k) sum += hist[k * nshells + s];
    out[s] = sum;
  }
}

// shell_sum[field][shell] += the blocks' partials (4 strided parts, then the parts
// in order), the new sums also into host memory, where the readbacks of a
// sample's ten fields find them without a launch each.  Block (64 shells,
// field), 256 threads.
__global__ void __launch_bounds__(256) sk_reduce_kernel(const double* __restrict__ partial, uint32_t blocks,
                                                        uint32_t nshells, double* __restrict__ shell_sum,
                                                        double* __restrict__ host_sum) {
  __shared__ double part[4][64];
  const uint32_t i = threadIdx.x & 63u, q = threadIdx.x >> 6, s = blockIdx.x * 64 + i;
  double acc = 0.0;
  if (s < nshells) {
    const double* col = partial + static_cast<size_t>(blockIdx.y) * blocks * nshells + s;
#pragma unroll 8
    for (uint32_t b = q; b < blocks; b += 4) acc += col[static_cast<size_t>(b) * nshells];
  }
  part[q][i] = acc;
  __syncthreads();
  if (q == 0 && s < nshells) {
    const size_t at = static_cast<size_t>(blockIdx.y) * nshells + s;
    const double sum = shell_sum[at] + (part[0][i] + part[1][i] + part[2][i] + part[3][i]);
    shell_sum[at] = sum;
    host_sum[at] = sum;
  }
}

// Wavevectors per shell.
__global__ void __launch_bounds__(256) sk_count_kernel(uint32_t nx, uint32_t ny, uint32_t nz, uint32_t nshells,
                                                       unsigned long long* __restrict__ shell_count) {
  extern __shared__ unsigned long long cnt[];
  for (uint32_t s = threadIdx.x; s < nshells; s += blockDim.x) cnt[s] = 0ull;
  __syncthreads();
  const uint32_t hx = nx / 2 + 1;
  for (uint32_t row = blockIdx.x; row < ny * nz; row += gridDim.x) {
    const uint32_t kz = row / ny, ky = row - kz * ny;
    const uint64_t kyz2 = static_cast<uint64_t>(wave2(ky, ny)) + wave2(kz, nz);
    for (uint32_t kx = threadIdx.x; kx < hx; kx += blockDim.x) {
      const uint64_t k2 = kyz2 + static_cast<uint64_t>(kx) * kx;
      if (k2 == 0) continue;
      const uint32_t shell = static_cast<uint32_t>(llrint(sqrt(static_cast<double>(k2))));
      if (shell < nshells) atomicAdd(&cnt[shell], kx == 0 || 2 * kx == nx ? 1ull : 2ull);
    }
  }
  __syncthreads();
  for (uint32_t s = threadIdx.x; s < nshells; s += blockDim.x)
    if (cnt[s]) atomicAdd(&shell_count[s], cnt[s]);
}

// Copies n 8-byte words (into host memory that the GPU can write).
__global__ void __launch_bounds__(256) sk_copy_kernel(const unsigned long long* __restrict__ src, uint32_t n,
                                                      unsigned long long* __restrict__ dst) {
  for (uint32_t i = blockIdx.x * 256 + threadIdx.x; i < n; i += gridDim.x * 256) dst[i] = src[i];
}

__global__ void sk_bin_kernel(const float2* __restrict__ spec, uint32_t nx, uint32_t ny, uint32_t nz,
                              uint32_t nshells, double inv_n, double* __restrict__ shell_sum) {
  extern __shared__ double sum[];
  for (uint32_t s = threadIdx.x; s < nshells; s += blockDim.x) sum[s] = 0.0;
  __syncthreads();
  const uint32_t hx = nx / 2 + 1;
  const uint64_t total = static_cast<uint64_t>(hx) * ny * nz;
  for (uint64_t e = blockIdx.x * static_cast<uint64_t>(blockDim.x) + threadIdx.x; e < total;
       e += static_cast<uint64_t>(gridDim.x) * blockDim.x) {
    const uint32_t kx = static_cast<uint32_t>(e % hx);
    const uint64_t r = e / hx;
    const uint32_t ky = static_cast<uint32_t>(r % ny);
    const uint32_t kz = static_cast<uint32_t>(r / ny);
    const int64_t sx = kx;
    const int64_t sy = ky <= ny / 2 ? static_cast<int64_t>(ky) : static_cast<int64_t>(ky) - ny;
    const int64_t sz = kz <= nz / 2 ? static_cast<int64_t>(kz) : static_cast<int64_t>(kz) - nz;
    const int64_t k2 = sx * sx + sy * sy + sz * sz;
    if (k2 == 0) continue;
    const uint32_t shell = static_cast<uint32_t>(llrint(sqrt(static_cast<double>(k2))));
    if (shell >= nshells) continue;
    const bool self_conj = kx == 0 || (nx % 2 == 0 && kx == nx / 2);
    const unsigned mult = self_conj ? 1u : 2u;
    const float2 c = spec[e];
    const double p = (static_cast<double>(c.x) * c.x + static_cast<double>(c.y) * c.y) * inv_n;
    atomicAdd(&sum[shell], p * mult);
  }
  __syncthreads();
  for (uint32_t s = threadIdx.x; s < nshells; s += blockDim.x)
    if (sum[s] != 0.0) atomicAdd(&shell_sum[s], sum[s]);
}


// Columns per tile and block size of the passes along an axis of length n:
// as many neighbouring columns (a power of two up to 64) as keep a thread at
// kFftPerThread values of a block of at most 512 threads.
SkTiles make_tiles(uint32_t n, uint32_t hx, uint64_t lines, uint64_t pitch) {
  SkTiles c{};
  c.hx = hx;
  c.lines = static_cast<uint32_t>(lines);
  c.pitch = pitch;
  while (c.log_tx < 6 && (n << (c.log_tx + 1)) <= 512 * kFftPerThread) ++c.log_tx;
  c.div_hx = make_fastdiv(hx);
  c.div_tx = c.log_tx > 0 ? make_fastdiv(1u << c.log_tx) : FastDiv{0u, 1u};
  const uint32_t need = ((n << c.log_tx) + kFftPerThread - 1) / kFftPerThread;
  c.threads = (need + 63) / 64 * 64;
  return c;
}

}  // namespace

uint32_t sk_blocks(uint32_t nx, uint32_t ny, uint32_t nz) {
  const uint32_t hx = nx / 2 + 1;
  const SkTiles c = make_tiles(nz, hx, static_cast<uint64_t>(ny) * hx, 0);
  const uint32_t tiles = (c.lines + (1u << c.log_tx) - 1) >> c.log_tx;
  const uint32_t per = (tiles + kSkBlocks - 1) / kSkBlocks;  // tiles a block walks
  return (tiles + per - 1) / per;
}

hipError_t launch_sk(int storage, const GatherArgs& g, const float2* twiddle, uint32_t nshells, float2* spec,
                     double* partial, double* shell_sum, double* host_sum, hipStream_t s) {
  if (!sk_fits(g.nx, g.ny, g.nz)) return hipErrorInvalidValue;
  const uint32_t hx = g.nx / 2 + 1;
  const uint64_t pitch = static_cast<uint64_t>(hx) * g.ny * g.nz;
  FftPlan px = make_fft_plan(g.nx), py = make_fft_plan(g.ny), pz = make_fft_plan(g.nz);
  px.twiddle = twiddle;
  py.twiddle = twiddle + g.nx;
  pz.twiddle = twiddle + g.nx + g.ny;
  SkRows r{};
  r.pairs = g.nx >= 256 ? 1 : 256 / g.nx;
  r.pitch = pitch;
  r.div_lines = make_fastdiv(kHalf * r.pairs);
  r.div_hx = make_fastdiv(hx);
  const uint32_t rows = g.ny * g.nz, row_threads = (r.pairs * g.nx + 63) / 64 * 64;
  const size_t row_lds = sizeof(float2) * (static_cast<size_t>(g.nx) * kHalf * r.pairs + g.nx);
  const dim3 row_grid((rows + 2 * r.pairs - 1) / (2 * r.pairs)), row_block(row_threads);
  const auto with_kind = [](const FftPlan& p, auto f) {
    switch (fft_kind(p)) {
      case kFftPow2: f(std::integral_constant<int, kFftPow2>{}); break;
      case kFftSmooth: f(std::integral_constant<int, kFftSmooth>{}); break;
      default: f(std::integral_constant<int, kFftPrimes>{}); break;
    }
  };
  const auto rows_storage = [&](auto st) {
    constexpr int S = decltype(st)::value;
    with_kind(px, [&](auto kind) {
      constexpr int K = decltype(kind)::value;
      hipLaunchKernelGGL((g.odd ? sk_rows_kernel<S, true, K> : sk_rows_kernel<S, false, K>), row_grid, row_block,
                         row_lds, s, g, px, r, spec);
    });
  };
  switch (storage) {
    case kF32: rows_storage(std::integral_constant<int, kF32>{}); break;
    case kF16: rows_storage(std::integral_constant<int, kF16>{}); break;
    case kBF16: rows_storage(std::integral_constant<int, kBF16>{}); break;
    default: return hipErrorInvalidValue;
  }
  const SkTiles cy = make_tiles(g.ny, hx, static_cast<uint64_t>(g.nz) * hx, pitch);
  const uint32_t y_tiles = (cy.lines + (1u << cy.log_tx) - 1) >> cy.log_tx;
  const uint32_t y_blocks = (y_tiles + 7) / 8 * 8;
  with_kind(py, [&](auto kind) {
    hipLaunchKernelGGL(sk_columns_kernel<decltype(kind)::value>, dim3(y_blocks, 10), dim3(cy.threads),
                       sizeof(float2) * ((static_cast<size_t>(g.ny) << cy.log_tx) + g.ny), s, py, cy, spec);
  });
  const SkTiles cz = make_tiles(g.nz, hx, static_cast<uint64_t>(g.ny) * hx, pitch);
  const uint32_t blocks = sk_blocks(g.nx, g.ny, g.nz);
  const uint32_t log_copies = nshells <= 512 ? 2 : 1;
  with_kind(pz, [&](auto kind) {
    hipLaunchKernelGGL(sk_shells_kernel<decltype(kind)::value>, dim3(blocks, 10), dim3(cz.threads),
                       sizeof(float2) * ((static_cast<size_t>(g.nz) << cz.log_tx) + g.nz) +
                           sizeof(double) * (static_cast<size_t>(nshells) << log_copies),
                       s, pz, cz, g.nx, g.ny, nshells, log_copies, 1.0 / (static_cast<double>(g.nx) * g.ny * g.nz),
                       static_cast<const float2*>(spec), partial);
  });
  hipLaunchKernelGGL(sk_reduce_kernel, dim3((nshells + 63) / 64, 10), dim3(256), 0, s,
                     static_cast<const double*>(partial), blocks, nshells, shell_sum, host_sum);
  return hipGetLastError();
}

hipError_t launch_sk_count(uint32_t nx, uint32_t ny, uint32_t nz, uint32_t nshells, unsigned long long* shell_count,
                           hipStream_t s) {
  const uint64_t rows = static_cast<uint64_t>(ny) * nz;
  hipLaunchKernelGGL(sk_count_kernel, dim3(static_cast<uint32_t>(rows < 1024 ? rows : 1024)), dim3(256),
                     static_cast<size_t>(nshells) * sizeof(unsigned long long), s, nx, ny, nz, nshells, shell_count);
  return hipGetLastError();
}

hipError_t launch_sk_copy(const void* src, uint32_t n, void* dst, hipStream_t s) {
  hipLaunchKernelGGL(sk_copy_kernel, dim3((n + 255) / 256), dim3(256), 0, s,
                     static_cast<const unsigned long long*>(src), n, static_cast<unsigned long long*>(dst));
  return hipGetLastError();
}

hipError_t launch_sk_bin(const void* spec, uint32_t nx, uint32_t ny, uint32_t nz, uint32_t nshells,
                         double* shell_sum, hipStream_t s) {
  const uint64_t total = static_cast<uint64_t>(nx / 2 + 1) * ny * nz;
  uint64_t blocks = (total + 255) / 256;
  if (blocks > 2048) blocks = 2048;
  hipLaunchKernelGGL(sk_bin_kernel, dim3(static_cast<uint32_t>(blocks)), dim3(256),
                     static_cast<size_t>(nshells) * sizeof(double), s, static_cast<const float2*>(spec), nx, ny, nz,
                     nshells, 1.0 / (static_cast<double>(nx) * ny * nz), shell_sum);
  return hipGetLastError();
}

}  // namespace rflbm

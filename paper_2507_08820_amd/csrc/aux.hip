// aux.hip -- kernels around the step: population readback and write-back in the
// canonical FP64 layout, equilibrium initialisation (Eq. hermite_feq2 in its
// product form), moment fields rho, j, Pi (Eqs. eq:rho, eq:u and the Pi of
// Sec. III), re-encoding of stored deviations, the noise generator exposed for
// testing, and a plain copy kernel (bandwidth reference).
//
// All of these work on the AA layout described in kernels.hpp: at an even step
// count f_i(x) sits in slot A[i][x], at an odd one in A[26 - i][x - c_i].
#include <hip/hip_runtime.h>

#include <type_traits>

#include "d3q27.hpp"
#include "kernels.hpp"
#include "philox.hpp"
#include "policy.hpp"
#include "slots.hpp"
#include "storage.hpp"

namespace rflbm {

namespace {

// Index of this thread in a launch over node_grid (policy.hpp).
__device__ __forceinline__ uint64_t thread_of_nodes() {
  return (blockIdx.x + blockIdx.y * kNodeGridX) * 256 + threadIdx.x;
}

dim3 node_blocks(uint64_t nodes) {
  const NodeGrid g = node_grid(nodes);
  return dim3(g.x, g.y);
}

// f(x, t) of every node, FP64 planar.  Bound by memory: 27 stored words in, 27
// FP64 values out a node.  One thread per node, whose 27 loads are in flight
// together; the outputs are streamed (non-temporal), since they are twice to
// four times the populations and only push those out of the caches.  192^3
// FP32 0.51 -> 0.43 ms, 256^3 FP16 1.24 -> 0.83 ms (6.6 TB/s copy rate: 0.35
// and 0.69); one population per block instead of 27 per thread took 0.49 and
// 1.09 ms.
template <int S, bool ODD>
__global__ void __launch_bounds__(256) get_pop_kernel(const GatherArgs g, double* __restrict__ dst) {
  using C = Codec<S>;
  using T = typename C::T;
  const uint32_t N = g.nx * g.ny * g.nz;
  const T* pop = static_cast<const T*>(g.pop);
  const uint64_t n64 = thread_of_nodes();
  if (n64 >= N) return;
  const uint32_t n = static_cast<uint32_t>(n64);
  const Slots<ODD> slot(coords32(n, g), g);
#pragma unroll
  for (int i = 0; i < kQ; ++i) {
    const int cls = speed_class(i);
    const float d = C::decode(pop[slot(i)], g.sigma[cls]);
    const double v = class_weight(cls) * g.rho0 + static_cast<double>(d);
    __builtin_nontemporal_store(v, dst + static_cast<uint64_t>(i) * N + n);
  }
}

template <int S>
__global__ void get_pop_at_kernel(const GatherArgs g, const uint32_t* nodes, uint32_t count, double* dst) {
  using C = Codec<S>;
  using T = typename C::T;
  const T* pop = static_cast<const T*>(g.pop);
  const uint32_t k = blockIdx.x * blockDim.x + threadIdx.x;
  if (k >= count) return;
  const uint32_t n = nodes[k];
  if (static_cast<uint64_t>(n) >= static_cast<uint64_t>(g.nx) * g.ny * g.nz) {
    // not a node of the box: nothing is read, the 27 values are NaN
#pragma unroll
    for (int i = 0; i < kQ; ++i) dst[static_cast<uint64_t>(i) * count + k] = __builtin_nan("");
    return;
  }
  const NodeXYZ p = coords(n, g.nx, g.ny);
#pragma unroll
  for (int i = 0; i < kQ; ++i) {
    const int cls = speed_class(i);
    const float d = C::decode(pop[slot_index(i, p, g)], g.sigma[cls]);
    dst[static_cast<uint64_t>(i) * count + k] = class_weight(cls) * g.rho0 + static_cast<double>(d);
  }
}

template <int S>
__global__ void set_pop_kernel(const GatherArgs g, const double* src) {
  using C = Codec<S>;
  using T = typename C::T;
  const uint64_t N = static_cast<uint64_t>(g.nx) * g.ny * g.nz;
  T* pop = static_cast<T*>(const_cast<void*>(g.pop));
  for (uint64_t n = blockIdx.x * static_cast<uint64_t>(blockDim.x) + threadIdx.x; n < N;
       n += static_cast<uint64_t>(gridDim.x) * blockDim.x) {
    const NodeXYZ p = coords(n, g.nx, g.ny);
#pragma unroll
    for (int i = 0; i < kQ; ++i) {
      const int cls = speed_class(i);
      const double d = src[i * N + n] - class_weight(cls) * g.rho0;
      pop[slot_index(i, p, g)] = C::encode(static_cast<float>(d), g.inv_sigma[cls]);
    }
  }
}

// f^(0)_i = rho prod_a omega(c_a) [1 + c_a u_a / cs2 + (c_a^2 - cs2) u_a^2 / (2 cs2^2)],
// the product form of the full-Hermite equilibrium (every Table II mode is a
// product of 1-D Hermite polynomials, so its Hermite sum factorises by axis).
template <int S>
__global__ void init_eq_kernel(const GatherArgs g, const double* rho, const double* u) {
  using C = Codec<S>;
  using T = typename C::T;
  const uint64_t N = static_cast<uint64_t>(g.nx) * g.ny * g.nz;
  T* pop = static_cast<T*>(const_cast<void*>(g.pop));
  for (uint64_t n = blockIdx.x * static_cast<uint64_t>(blockDim.x) + threadIdx.x; n < N;
       n += static_cast<uint64_t>(gridDim.x) * blockDim.x) {
    const NodeXYZ p = coords(n, g.nx, g.ny);
    const double r = rho ? rho[n] : g.rho0;
    const double ua[3] = {u ? u[n] : 0.0, u ? u[N + n] : 0.0, u ? u[2 * N + n] : 0.0};
    double fac[3][3];  // fac[a][c + 1]
#pragma unroll
    for (int a = 0; a < 3; ++a) {
      const double q = 4.5 * ua[a] * ua[a];
      fac[a][0] = (1.0 / 6.0) * (1.0 - 3.0 * ua[a] + q - 1.5 * ua[a] * ua[a]);
      fac[a][1] = (2.0 / 3.0) * (1.0 - 1.5 * ua[a] * ua[a]);
      fac[a][2] = (1.0 / 6.0) * (1.0 + 3.0 * ua[a] + q - 1.5 * ua[a] * ua[a]);
    }
#pragma unroll
    for (int i = 0; i < kQ; ++i) {
      const int cls = speed_class(i);
      const double feq = r * fac[0][i % 3] * fac[1][(i / 3) % 3] * fac[2][i / 9];
      const double d = feq - class_weight(cls) * g.rho0;
      pop[slot_index(i, p, g)] = C::encode(static_cast<float>(d), g.inv_sigma[cls]);
    }
  }
}

// cos and sin of 2 pi a / 65536, a in 0 .. 65535, in FP64: a = 16384 q + r with
// |r| <= 8192 exactly, then the Taylor series on |theta| <= pi / 4 (the first
// terms left out, theta^18 / 18! and theta^19 / 19!, are below 3e-18).
__device__ __forceinline__ void cos_sin_turn16(uint32_t a, double& c, double& s) {
  const uint32_t q = (a + 8192u) >> 14;
  const double th = static_cast<double>(static_cast<int>(a) - static_cast<int>(q << 14)) *
                    (6.283185307179586476925 / 65536.0);
  const double t2 = th * th;
  double cp = 1.0 / 20922789888000.0, sp = 1.0 / 355687428096000.0;  // 1/16!, 1/17!
  cp = fma(cp, t2, -1.0 / 87178291200.0);
  sp = fma(sp, t2, -1.0 / 1307674368000.0);
  cp = fma(cp, t2, 1.0 / 479001600.0);
  sp = fma(sp, t2, 1.0 / 6227020800.0);
  cp = fma(cp, t2, -1.0 / 3628800.0);
  sp = fma(sp, t2, -1.0 / 39916800.0);
  cp = fma(cp, t2, 1.0 / 40320.0);
  sp = fma(sp, t2, 1.0 / 362880.0);
  cp = fma(cp, t2, -1.0 / 720.0);
  sp = fma(sp, t2, -1.0 / 5040.0);
  cp = fma(cp, t2, 1.0 / 24.0);
  sp = fma(sp, t2, 1.0 / 120.0);
  cp = fma(cp, t2, -0.5);
  sp = fma(sp, t2, -1.0 / 6.0);
  const double cr = fma(cp, t2, 1.0);
  const double sr = fma(th * t2, sp, th);
  // rotate by q quarter turns
  const double ca = (q & 1u) ? sr : cr, sa = (q & 1u) ? cr : sr;
  c = ((q + 1u) & 2u) ? -ca : ca;
  s = (q & 2u) ? -sa : sa;
}

// ln(k 2^-23) for k in 1 .. 2^23, in FP64: k = m 2^e with m in [sqrt(1/2), sqrt(2)),
// ln m = 2 atanh(s) with s = (m - 1) / (m + 1), |s| < 0.1716, by its Taylor
// series (the first term left out, s^20 / 21 of the sum, is below 3e-17).
__device__ __forceinline__ double log_k23(uint32_t k) {
  const double x = static_cast<double>(k);
  double m = __builtin_amdgcn_frexp_mant(x);  // [1/2, 1)
  int e = __builtin_amdgcn_frexp_exp(x);
  const bool low = m < 0.70710678118654752440;
  m = low ? m + m : m;
  e = (low ? e - 1 : e) - 23;
  const double num = m - 1.0, den = m + 1.0;
  double rc = __builtin_amdgcn_rcp(den);
  rc = fma(rc, fma(-den, rc, 1.0), rc);
  rc = fma(rc, fma(-den, rc, 1.0), rc);
  double s = num * rc;
  s = fma(rc, fma(-den, s, num), s);
  const double s2 = s * s;
  double p = 1.0 / 19.0;
  p = fma(p, s2, 1.0 / 17.0);
  p = fma(p, s2, 1.0 / 15.0);
  p = fma(p, s2, 1.0 / 13.0);
  p = fma(p, s2, 1.0 / 11.0);
  p = fma(p, s2, 1.0 / 9.0);
  p = fma(p, s2, 1.0 / 7.0);
  p = fma(p, s2, 1.0 / 5.0);
  p = fma(p, s2, 1.0 / 3.0);
  // ln 2 = hi + lo, hi with 32 bits, so that e hi is exact
  constexpr double kLn2Hi = 0x1.62e42fefp-1, kLn2Lo = 0x1.473de6af278edp-34;
  const double ed = static_cast<double>(e), t = s + s;
  return fma(ed, kLn2Hi, fma(t * s2, p, fma(ed, kLn2Lo, t)));
}

// Thermalised start: f_i = f^(0)_i(rho, u) + sqrt(rho0 kT w_i / cs2) xi_i, the
// stationary covariance of the fluctuating update (Eq. fluct_phi) in the
// linear regime.  xi_i is normal i of the node's Box-Muller stream at the
// reserved step word 0xFFFFFFFF, Philox calls j = 0..4 (30 normals, 27 used);
// set-up code, so the transform runs in FP64.
//
// Bound by FP64 issue.  Each pair of normals goes straight into its two
// populations, so a lane holds one pair at a time, and the angle, a 16-bit
// integer, needs no argument reduction.  192^3 FP32: 0.39 ms, 930 FP64
// instructions a node; with the library's log, cos and sin on FP64 arguments and
// all 30 normals held at once it took 2.08 ms (772 bytes of scratch a lane).
template <int S, int R, bool ODD>
__global__ void __launch_bounds__(256) init_thermal_kernel(const GatherArgs g, const double* rho, const double* u,
                                                           uint32_t key0, uint32_t key1, uint32_t sid, double kT) {
  using C = Codec<S>;
  using T = typename C::T;
  const uint32_t N = g.nx * g.ny * g.nz;
  T* pop = static_cast<T*>(const_cast<void*>(g.pop));
  const double mu = g.rho0 * kT * 3.0;
  const uint64_t n64 = thread_of_nodes();
  if (n64 >= N) return;
  const uint32_t n = static_cast<uint32_t>(n64);
  const Slots<ODD> slot(coords32(n, g), g);
  const double r = rho ? rho[n] : g.rho0;
  const uint64_t N1 = N, N2 = 2 * N1;
  const double ua[3] = {u ? u[n] : 0.0, u ? u[N1 + n] : 0.0, u ? u[N2 + n] : 0.0};
  double fac[3][3];
#pragma unroll
  for (int a = 0; a < 3; ++a) {
    const double uu = ua[a] * ua[a];
    fac[a][0] = (1.0 / 6.0) * (1.0 - 3.0 * ua[a] + 3.0 * uu);
    fac[a][1] = (2.0 / 3.0) * (1.0 - 1.5 * uu);
    fac[a][2] = (1.0 / 6.0) * (1.0 + 3.0 * ua[a] + 3.0 * uu);
  }
  double amp[4];  // sqrt(mu w) per speed class
#pragma unroll
  for (int cls = 0; cls < 4; ++cls) amp[cls] = sqrt(mu * class_weight(cls));
#pragma unroll
  for (int j = 0; j < 5; ++j) {
    const Word4 w = philox<R>(Word4{n, 0xFFFFFFFFu, static_cast<uint32_t>(j), sid}, key0, key1);
    // pair m: radius uniform 1 - (w_m >> 9) 2^-23, angle uniform a_m 2^-16
    const uint32_t wr[3] = {w.w0, w.w1, w.w2};
    const uint32_t am[3] = {w.w3 >> 16, w.w3 & 0xFFFFu, ((w.w0 & 0xFFu) << 8) | (w.w1 & 0xFFu)};
#pragma unroll
    for (int m = 0; m < 3; ++m) {
      const int i0 = 6 * j + 2 * m;  // normals i0, i0 + 1 go to populations i0, i0 + 1
      if (i0 >= kQ) continue;
      const double rad = sqrt(-2.0 * log_k23((1u << 23) - (wr[m] >> 9)));
      double z[2];
      cos_sin_turn16(am[m], z[0], z[1]);
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        const int i = i0 + h;
        if (i >= kQ) continue;
        const int cls = speed_class(i);
        const double feq = r * fac[0][i % 3] * fac[1][(i / 3) % 3] * fac[2][i / 9];
        const double d = feq - class_weight(cls) * g.rho0 + amp[cls] * (rad * z[h]);
        pop[slot(i)] = C::encode(static_cast<float>(d), g.inv_sigma[cls]);
      }
    }
  }
}

// Moment fields of the nodes n0 .. n0 + count - 1: field c of node n0 + k goes
// to dst[c * pitch + k].
// NT: populations read past the caches (read_streams, policy.hpp).
template <int S, bool ODD, bool NT>
__global__ void __launch_bounds__(256) moments_kernel(const GatherArgs g, uint32_t mask, uint64_t n0, uint64_t count,
                                                      uint64_t pitch, float* __restrict__ dst) {
  using C = Codec<S>;
  using T = typename C::T;
  const T* pop = static_cast<const T*>(g.pop);
  const uint64_t k = thread_of_nodes();
  if (k >= count) return;
  const Slots<ODD> slot(coords32(static_cast<uint32_t>(n0 + k), g), g);
  float v[kQ];
#pragma unroll
  for (int i = 0; i < kQ; ++i) {
    const T q = NT ? __builtin_nontemporal_load(pop + slot(i)) : pop[slot(i)];
    v[i] = C::decode(q, g.sigma[speed_class(i)]);
  }
  forward27(v);
  float* out = dst;
  auto put = [&](uint64_t at, float q) {
    if constexpr (NT) __builtin_nontemporal_store(q, out + at);
    else out[at] = q;
  };
  if (mask & 1u) {
    put(k, static_cast<float>(g.rho0 + static_cast<double>(v[0])));
    out += pitch;
  }
  if (mask & 2u) {
    put(k, v[1]);
    put(pitch + k, v[3]);
    put(2 * pitch + k, v[9]);
    out += 3 * pitch;
  }
  if (mask & 4u) {
    const int slots[6] = {mode_slot(4), mode_slot(5), mode_slot(6), mode_slot(7), mode_slot(8), mode_slot(9)};
#pragma unroll
    for (int c = 0; c < 6; ++c) put(c * pitch + k, v[slots[c]]);
  }
}

// Slot A[p][.] holds populations of one speed class at either parity (26 - i
// and i have the same |c|^2), so re-encoding works slot by slot.
template <int S>
__global__ void reencode_kernel(const GatherArgs from, const GatherArgs to) {
  using C = Codec<S>;
  using T = typename C::T;
  const uint64_t N = static_cast<uint64_t>(from.nx) * from.ny * from.nz;
  T* pop = static_cast<T*>(const_cast<void*>(from.pop));
  const uint64_t total = N * kQ;
  for (uint64_t e = blockIdx.x * static_cast<uint64_t>(blockDim.x) + threadIdx.x; e < total;
       e += static_cast<uint64_t>(gridDim.x) * blockDim.x) {
    // e runs over (x, plane, y, z) with x fastest; padding is left untouched
    const uint32_t x = static_cast<uint32_t>(e % from.nx);
    const uint64_t r = e / from.nx;
    const int plane = static_cast<int>(r % kQ);
    const uint64_t row = r / kQ;
    const int cls = speed_class(plane);
    T* q = pop + element_index(plane, x, static_cast<uint32_t>(row % from.ny),
                               static_cast<uint32_t>(row / from.ny), from);
    const double d = static_cast<double>(C::decode(*q, from.sigma[cls])) +
                     class_weight(cls) * (from.rho0 - to.rho0);
    *q = C::encode(static_cast<float>(d), to.inv_sigma[cls]);
  }
}

template <int R>
__global__ void rng_kernel(uint32_t key0, uint32_t key1, uint32_t sid, uint32_t node0, uint32_t count,
                           uint32_t step, float* u, float* z) {
  const uint32_t t = blockIdx.x * blockDim.x + threadIdx.x;
  if (t >= count) return;
  const uint32_t node = node0 + t;
#pragma unroll
  for (uint32_t j = 0; j < 4; ++j) {
    const Word4 w = philox<R>(Word4{node, step, j, sid}, key0, key1);
    float r[6], uu[6];
    box_muller<0>(w, r[0], r[1]);
    box_muller<1>(w, r[2], r[3]);
    box_muller<2>(w, r[4], r[5]);
    uu[0] = radius_uniform(w.w0);
    uu[1] = angle_uniform<0>(w);
    uu[2] = radius_uniform(w.w1);
    uu[3] = angle_uniform<1>(w);
    uu[4] = radius_uniform(w.w2);
    uu[5] = angle_uniform<2>(w);
#pragma unroll
    for (int q = 0; q < 6; ++q) {
      u[static_cast<uint64_t>(t) * 24 + 6 * j + q] = uu[q];
      z[static_cast<uint64_t>(t) * 24 + 6 * j + q] = r[q];
    }
  }
}

typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));

// One 16-byte vector per thread, non-temporal loads and stores: the fastest
// of the copy forms measured on MI355X (one to eight vectors per thread,
// with and without non-temporal hints).
__global__ void __launch_bounds__(256) copy_kernel(u32x4* __restrict__ dst, const u32x4* __restrict__ src,
                                                   uint64_t n) {
  const uint64_t e = static_cast<uint64_t>(blockIdx.x) * 256 + threadIdx.x;
  if (e < n) __builtin_nontemporal_store(__builtin_nontemporal_load(src + e), dst + e);
}

__global__ void fill_zero_kernel(double* dst, uint64_t n) {
  for (uint64_t e = blockIdx.x * static_cast<uint64_t>(blockDim.x) + threadIdx.x; e < n;
       e += static_cast<uint64_t>(gridDim.x) * blockDim.x)
    dst[e] = 0.0;
}

__global__ void set_u32_kernel(uint32_t* dst, uint32_t value) {
  if (threadIdx.x == 0) *dst = value;
}

// Parity change of the stored state.  The slot of f_j(y) at the new parity is
// A'[j][y] = A[26 - j][y - c_j] of the old one, in either direction; read for
// 26 - j at y - c_j it says A'[26 - j][y - c_j] = A[j][y], so the two slots
// simply exchange their stored words (the rest population stays).  One thread
// per node swaps its 13 pairs, which no other thread touches: in place, bit for
// bit, no scratch.  Bound by memory (52 words a node).  In a restart of 128 x 112
// x 96 FP16 it replaced 39 launches through a scratch plane (0.27 ms) and that
// plane's allocation: 0.70 -> 0.31 ms in all, with faster readbacks 0.02 of it.
template <typename W>
__global__ void __launch_bounds__(256) swap_parity_kernel(const GatherArgs g) {
  const uint32_t N = g.nx * g.ny * g.nz;
  W* pop = static_cast<W*>(const_cast<void*>(g.pop));
  const uint64_t n = thread_of_nodes();
  if (n >= N) return;
  const Slots<true> slot(coords32(static_cast<uint32_t>(n), g), g);
  const uint64_t own = slot.row[4] + slot.xs[1];
  W a[kQ / 2], b[kQ / 2];
#pragma unroll
  for (int j = 0; j < kQ / 2; ++j) {
    a[j] = pop[own + static_cast<uint32_t>(j) * slot.pitch];
    b[j] = pop[slot(j)];
  }
#pragma unroll
  for (int j = 0; j < kQ / 2; ++j) {
    pop[own + static_cast<uint32_t>(j) * slot.pitch] = b[j];
    pop[slot(j)] = a[j];
  }
}

uint32_t grid_for(uint64_t work, uint32_t block) {
  const uint64_t g = (work + block - 1) / block;
  return static_cast<uint32_t>(g < 65536 ? (g == 0 ? 1 : g) : 65536);
}

}  // namespace

#define RFLBM_DISPATCH_STORAGE(storage, KERNEL, grid, block, stream, ...)                  \
  do {                                                                                      \
    switch (storage) {                                                                      \
      case kF32: hipLaunchKernelGGL(KERNEL<kF32>, grid, block, 0, stream, __VA_ARGS__); break;   \
      case kF16: hipLaunchKernelGGL(KERNEL<kF16>, grid, block, 0, stream, __VA_ARGS__); break;   \
      case kBF16: hipLaunchKernelGGL(KERNEL<kBF16>, grid, block, 0, stream, __VA_ARGS__); break; \
      default: return hipErrorInvalidValue;                                                 \
    }                                                                                       \
  } while (0)

// Calls f(integral_constant<int, S>) for the storage type; the launch error, if any.
template <class F>
hipError_t with_storage(int storage, F f) {
  switch (storage) {
    case kF32: f(std::integral_constant<int, kF32>{}); break;
    case kF16: f(std::integral_constant<int, kF16>{}); break;
    case kBF16: f(std::integral_constant<int, kBF16>{}); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

hipError_t launch_get_populations(int storage, const GatherArgs& g, double* dst, hipStream_t s) {
  const uint64_t N = static_cast<uint64_t>(g.nx) * g.ny * g.nz;
  const dim3 grid = node_blocks(N), block(256);
  return with_storage(storage, [&](auto st) {
    constexpr int S = decltype(st)::value;
    if (g.odd) hipLaunchKernelGGL((get_pop_kernel<S, true>), grid, block, 0, s, g, dst);
    else hipLaunchKernelGGL((get_pop_kernel<S, false>), grid, block, 0, s, g, dst);
  });
}

hipError_t launch_get_populations_at(int storage, const GatherArgs& g, const uint32_t* nodes, uint32_t count,
                                     double* dst, hipStream_t s) {
  if (count == 0) return hipSuccess;
  RFLBM_DISPATCH_STORAGE(storage, get_pop_at_kernel, dim3((count + 255) / 256), dim3(256), s, g, nodes, count, dst);
  return hipGetLastError();
}

hipError_t launch_set_populations(int storage, const GatherArgs& g, const double* src, hipStream_t s) {
  const uint64_t N = static_cast<uint64_t>(g.nx) * g.ny * g.nz;
  RFLBM_DISPATCH_STORAGE(storage, set_pop_kernel, dim3(grid_for(N, 256)), dim3(256), s, g, src);
  return hipGetLastError();
}

hipError_t launch_init_equilibrium(int storage, const GatherArgs& g, const double* rho,
                                   const double* u, hipStream_t s) {
  const uint64_t N = static_cast<uint64_t>(g.nx) * g.ny * g.nz;
  RFLBM_DISPATCH_STORAGE(storage, init_eq_kernel, dim3(grid_for(N, 256)), dim3(256), s, g, rho, u);
  return hipGetLastError();
}

hipError_t launch_init_thermal(int storage, const GatherArgs& g, const double* rho, const double* u,
                               uint32_t key0, uint32_t key1, uint32_t sid, int rounds, double kT,
                               hipStream_t s) {
  const uint64_t N = static_cast<uint64_t>(g.nx) * g.ny * g.nz;
  const dim3 grid = node_blocks(N), block(256);
  if (rounds != 7 && rounds != 10) return hipErrorInvalidValue;
  return with_storage(storage, [&](auto st) {
    constexpr int S = decltype(st)::value;
    const auto go = [&](auto kernel) { hipLaunchKernelGGL(kernel, grid, block, 0, s, g, rho, u, key0, key1, sid, kT); };
    if (rounds == 7) go(g.odd ? init_thermal_kernel<S, 7, true> : init_thermal_kernel<S, 7, false>);
    else go(g.odd ? init_thermal_kernel<S, 10, true> : init_thermal_kernel<S, 10, false>);
  });
}

hipError_t launch_get_moments(int storage, const GatherArgs& g, uint32_t mask, float* dst,
                              hipStream_t s) {
  const uint64_t N = static_cast<uint64_t>(g.nx) * g.ny * g.nz;
  return launch_get_moments_range(storage, g, mask, 0, N, dst, N, s);
}

hipError_t launch_get_moments_range(int storage, const GatherArgs& g, uint32_t mask, uint64_t n0,
                                    uint64_t count, float* dst, uint64_t pitch, hipStream_t s) {
  if (count == 0) return hipSuccess;
  const dim3 grid = node_blocks(count), block(256);
  const uint64_t pop_bytes = static_cast<uint64_t>(kQ) * g.nx * g.ny * g.nz * storage_bytes(storage);
  const bool nt = read_streams(static_cast<uint64_t>(g.nx) * storage_bytes(storage), pop_bytes, g.odd != 0);
  return with_storage(storage, [&](auto st) {
    constexpr int S = decltype(st)::value;
    const auto kernel = g.odd ? moments_kernel<S, true, false>
                              : (nt ? moments_kernel<S, false, true> : moments_kernel<S, false, false>);
    hipLaunchKernelGGL(kernel, grid, block, 0, s, g, mask, n0, count, pitch, dst);
  });
}

hipError_t launch_reencode(int storage, const GatherArgs& from, const GatherArgs& to, hipStream_t s) {
  const uint64_t N = static_cast<uint64_t>(from.nx) * from.ny * from.nz;
  RFLBM_DISPATCH_STORAGE(storage, reencode_kernel, dim3(grid_for(N * kQ, 256)), dim3(256), s, from, to);
  return hipGetLastError();
}

hipError_t launch_rng_normals(uint32_t key0, uint32_t key1, uint32_t stream_id, int rounds,
                              uint32_t node0, uint32_t count, uint32_t step, float* u, float* z,
                              hipStream_t s) {
  const dim3 grid((count + 255) / 256), block(256);
  if (count == 0) return hipSuccess;
  if (rounds == 10)
    hipLaunchKernelGGL(rng_kernel<10>, grid, block, 0, s, key0, key1, stream_id, node0, count, step, u, z);
  else if (rounds == 7)
    hipLaunchKernelGGL(rng_kernel<7>, grid, block, 0, s, key0, key1, stream_id, node0, count, step, u, z);
  else
    return hipErrorInvalidValue;
  return hipGetLastError();
}

hipError_t launch_swap_parity(int storage, const GatherArgs& g, hipStream_t s) {
  const uint64_t N = static_cast<uint64_t>(g.nx) * g.ny * g.nz;
  const dim3 grid = node_blocks(N), block(256);
  if (storage_bytes(storage) == 4) hipLaunchKernelGGL(swap_parity_kernel<uint32_t>, grid, block, 0, s, g);
  else hipLaunchKernelGGL(swap_parity_kernel<uint16_t>, grid, block, 0, s, g);
  return hipGetLastError();
}

hipError_t launch_copy(void* dst, const void* src, size_t bytes, hipStream_t s) {
  const uint64_t n = bytes / sizeof(u32x4);
  if (n == 0) return hipSuccess;
  const uint64_t blocks = (n + 255) / 256;
  if (blocks > 0x7fffffffull) return hipErrorInvalidValue;
  hipLaunchKernelGGL(copy_kernel, dim3(static_cast<uint32_t>(blocks)), dim3(256), 0, s,
                     static_cast<u32x4*>(dst), static_cast<const u32x4*>(src), n);
  return hipGetLastError();
}

hipError_t launch_set_u32(uint32_t* dst, uint32_t value, hipStream_t s) {
  hipLaunchKernelGGL(set_u32_kernel, dim3(1), dim3(64), 0, s, dst, value);
  return hipGetLastError();
}

hipError_t launch_fill_zero(double* dst, size_t n, hipStream_t s) {
  if (n == 0) return hipSuccess;
  hipLaunchKernelGGL(fill_zero_kernel, dim3(grid_for(n, 256)), dim3(256), 0, s, dst,
                     static_cast<uint64_t>(n));
  return hipGetLastError();
}

}  // namespace rflbm

// fft.hpp -- lines of complex FP32 values transformed in LDS, for the structure
// factor (sk.hip): decimation in time by the self-sorting (Stockham) scheme,
// radices 8, 4, 2, 3, 5, 7 in registers, any other prime factor by its sum.
//
// A block holds `lines` lines of n values, value p of line l at lds[p * lines + l],
// so that neighbouring lanes work on neighbouring lines and every LDS access of
// a wave is contiguous.  One pass of radix r: task (j, l), j < n / r, reads the
// values j + q n / r, multiplies by the twiddles exp(-2 pi i q k / (Ns r)), k =
// j mod Ns (Ns: product of the earlier radices), transforms the r values and
// writes them to (j - k) r + k + q Ns.  All reads of a pass come before all
// writes, with the values in registers, so one buffer is enough (32 KiB where
// two would take 64: twice the blocks on a CU).
#pragma once
#include <cstdint>
#include <hip/hip_runtime.h>

#include "fastdiv.hpp"
#include "policy.hpp"

namespace rflbm {

constexpr int kFftMaxPasses = 12;
constexpr int kFftPerThread = 8;      // values a thread holds in a pass

struct FftPlan {
  uint32_t n;
  uint32_t passes;
  uint32_t radix[kFftMaxPasses];
  FastDiv div_ns[kFftMaxPasses];  // division by Ns (Ns >= 2)
  const float2* twiddle;          // exp(-2 pi i t / n), t < n (device memory)
};

// Radices of a transform of length n (twiddle left null).
inline FftPlan make_fft_plan(uint32_t n) {
  FftPlan p{};
  p.n = n;
  uint32_t left = n, ns = 1;
  const auto add = [&](uint32_t r) {
    p.radix[p.passes] = r;
    p.div_ns[p.passes] = ns >= 2 ? make_fastdiv(ns) : FastDiv{0u, 1u};
    ++p.passes;
    ns *= r;
    left /= r;
  };
  for (uint32_t r : {8u, 4u, 2u, 3u, 5u, 7u})
    while (left % r == 0) add(r);
  uint32_t r = 11;
  while (left > 1) {
    if (left % r == 0) add(r);
    else r += 2;
  }
  return p;
}

// What the passes of a transform need, for kernels compiled per kind (the passes
// left out free registers, hence waves): powers of two; radices up to 8; any.
enum FftKind : int { kFftPow2 = 0, kFftSmooth = 1, kFftPrimes = 2 };
inline FftKind fft_kind(const FftPlan& p) {
  const uint32_t last = p.passes > 0 ? p.radix[p.passes - 1] : 2u;  // the odd ones come last
  return last > 8 ? kFftPrimes : (last % 2 != 0 ? kFftSmooth : kFftPow2);
}

__device__ __forceinline__ float2 cmul(float2 a, float2 b) {
  return make_float2(fmaf(a.x, b.x, -(a.y * b.y)), fmaf(a.x, b.y, a.y * b.x));
}
__device__ __forceinline__ float2 cadd(float2 a, float2 b) { return make_float2(a.x + b.x, a.y + b.y); }
__device__ __forceinline__ float2 csub(float2 a, float2 b) { return make_float2(a.x - b.x, a.y - b.y); }
__device__ __forceinline__ float2 cmul_mi(float2 a) { return make_float2(a.y, -a.x); }  // -i a

// cos and sin of 2 pi k / r for r = 3, 5, 7, k = 1 .. (r - 1) / 2.
template <int R>
struct Roots;
template <>
struct Roots<3> {
  static constexpr float c[1] = {-0.5f}, s[1] = {0.86602540378443864676f};
};
template <>
struct Roots<5> {
  static constexpr float c[2] = {0.30901699437494742410f, -0.80901699437494742410f};
  static constexpr float s[2] = {0.95105651629515357212f, 0.58778525229247312917f};
};
template <>
struct Roots<7> {
  static constexpr float c[3] = {0.62348980185873353053f, -0.22252093395631440429f, -0.90096886790241912624f};
  static constexpr float s[3] = {0.78183148246802980871f, 0.97492791218182360702f, 0.43388373911755812048f};
};

// In-place DFT of R values.
template <int R>
__device__ __forceinline__ void dft(float2 (&v)[R]) {
  if constexpr (R == 2) {
    const float2 a = v[0];
    v[0] = cadd(a, v[1]);
    v[1] = csub(a, v[1]);
  } else if constexpr (R == 4) {
    const float2 a = cadd(v[0], v[2]), b = csub(v[0], v[2]), c = cadd(v[1], v[3]), d = cmul_mi(csub(v[1], v[3]));
    v[0] = cadd(a, c);
    v[1] = cadd(b, d);
    v[2] = csub(a, c);
    v[3] = csub(b, d);
  } else if constexpr (R == 8) {
    float2 e[4] = {v[0], v[2], v[4], v[6]}, o[4] = {v[1], v[3], v[5], v[7]};
    dft<4>(e);
    dft<4>(o);
    constexpr float h = 0.70710678118654752440f;
    o[1] = make_float2(h * (o[1].x + o[1].y), h * (o[1].y - o[1].x));
    o[2] = cmul_mi(o[2]);
    o[3] = make_float2(h * (o[3].y - o[3].x), -h * (o[3].x + o[3].y));
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      v[k] = cadd(e[k], o[k]);
      v[k + 4] = csub(e[k], o[k]);
    }
  } else {
    // odd prime: pairs (q, R - q) share cosine and sine
    constexpr int H = (R - 1) / 2;
    float2 a[H], b[H], sum = v[0];
#pragma unroll
    for (int q = 0; q < H; ++q) {
      a[q] = cadd(v[q + 1], v[R - 1 - q]);
      b[q] = csub(v[q + 1], v[R - 1 - q]);
      sum = cadd(sum, a[q]);
    }
    const float2 v0 = v[0];
    v[0] = sum;
#pragma unroll
    for (int k = 1; k <= H; ++k) {
      float2 re = v0, im = make_float2(0.0f, 0.0f);  // sums of cos a and of sin b
#pragma unroll
      for (int q = 1; q <= H; ++q) {
        const int t = (k * q) % R;
        const float c = Roots<R>::c[(t <= H ? t : R - t) - 1];
        const float s = t <= H ? Roots<R>::s[t - 1] : -Roots<R>::s[R - t - 1];
        re.x = fmaf(c, a[q - 1].x, re.x);
        re.y = fmaf(c, a[q - 1].y, re.y);
        im.x = fmaf(s, b[q - 1].x, im.x);
        im.y = fmaf(s, b[q - 1].y, im.y);
      }
      // e^{-i t} v: cos a - i sin b
      v[k] = make_float2(re.x + im.y, re.y - im.x);
      v[R - k] = make_float2(re.x - im.y, re.y + im.x);
    }
  }
}

// One pass of radix R over every line (see the file's head).
template <int R>
__device__ __forceinline__ void fft_pass(float2* lds, const float2* tw, uint32_t lines, FastDiv div_lines,
                                         const FftPlan& p, uint32_t ns, FastDiv div_ns, uint32_t tid,
                                         uint32_t nthreads) {
  constexpr int P = R >= 8 ? 1 : (kFftPerThread + R - 1) / R;  // tasks a thread holds
  const uint32_t m = p.n / R, tasks = m * lines, step = m / ns;
  float2 v[P][R];
  uint32_t out[P];
#pragma unroll
  for (int i = 0; i < P; ++i) {
    const uint32_t task = tid + i * nthreads;
    if (task < tasks) {
      const uint32_t j = div_by(task, lines, div_lines), l = task - j * lines;
      const uint32_t b = div_by(j, ns, div_ns), k = j - b * ns;
#pragma unroll
      for (int q = 0; q < R; ++q) v[i][q] = lds[task + q * m * lines];
      if (ns > 1) {
#pragma unroll
        for (int q = 1; q < R; ++q) v[i][q] = cmul(v[i][q], tw[q * k * step]);
      }
      dft<R>(v[i]);
      out[i] = (b * ns * R + k) * lines + l;
    }
  }
  __syncthreads();
#pragma unroll
  for (int i = 0; i < P; ++i) {
    if (tid + i * nthreads < tasks) {
#pragma unroll
      for (int q = 0; q < R; ++q) lds[out[i] + q * ns * lines] = v[i][q];
    }
  }
  __syncthreads();
}

// A pass whose radix is another prime: each output is its sum over the r inputs,
// in partial sums of 16 (one running sum of r terms would lose digits a short
// transform keeps).  A thread's outputs lie nthreads apart; where that is a
// whole number of output positions of one line, and the pass is the whole
// transform (r = n), they share every input read.
__device__ inline void fft_pass_prime(float2* lds, const float2* tw, uint32_t lines, FastDiv div_lines,
                                      const FftPlan& p, uint32_t r, uint32_t ns, FastDiv div_ns, uint32_t tid,
                                      uint32_t nthreads) {
  const uint32_t m = p.n / r, total = p.n * lines, step = m / ns;
  uint32_t in[kFftPerThread], turn[kFftPerThread], t[kFftPerThread];
  float2 v[kFftPerThread];
  bool shared_in = true;
#pragma unroll
  for (int i = 0; i < kFftPerThread; ++i) {
    const uint32_t e = tid + i * nthreads;
    const uint32_t o = div_by(e, lines, div_lines), l = e - o * lines;  // output position and line
    const uint32_t w = div_by(o, ns, div_ns), k = o - w * ns;           // o = (b r + q) ns + k
    const uint32_t b = w / r, q = w - b * r;
    const bool live = e < total;
    in[i] = live ? (b * ns + k) * lines + l : 0u;  // input s: in + s m lines
    turn[i] = live ? (k + q * ns) * step : 0u;     // and exp(-2 pi i s (k + q ns) / (ns r)), turn < n
    t[i] = 0;
    v[i] = make_float2(0.0f, 0.0f);
    shared_in = shared_in && (!live || in[i] == in[0]);
  }
  const uint32_t pitch = m * lines;
  for (uint32_t s0 = 0; s0 < r; s0 += 16) {
    float2 part[kFftPerThread];
#pragma unroll
    for (int i = 0; i < kFftPerThread; ++i) part[i] = make_float2(0.0f, 0.0f);
    const uint32_t s1 = s0 + 16 < r ? s0 + 16 : r;
    if (shared_in) {
      for (uint32_t s = s0; s < s1; ++s) {
        const float2 a = lds[in[0] + s * pitch];
#pragma unroll
        for (int i = 0; i < kFftPerThread; ++i) {
          const float2 c = tw[t[i]];
          part[i].x = fmaf(a.x, c.x, fmaf(-a.y, c.y, part[i].x));
          part[i].y = fmaf(a.x, c.y, fmaf(a.y, c.x, part[i].y));
          t[i] += turn[i];
          t[i] -= t[i] >= p.n ? p.n : 0u;
        }
      }
    } else {
      for (uint32_t s = s0; s < s1; ++s) {
#pragma unroll
        for (int i = 0; i < kFftPerThread; ++i) {
          const float2 a = lds[in[i] + s * pitch], c = tw[t[i]];
          part[i].x = fmaf(a.x, c.x, fmaf(-a.y, c.y, part[i].x));
          part[i].y = fmaf(a.x, c.y, fmaf(a.y, c.x, part[i].y));
          t[i] += turn[i];
          t[i] -= t[i] >= p.n ? p.n : 0u;
        }
      }
    }
#pragma unroll
    for (int i = 0; i < kFftPerThread; ++i) v[i] = cadd(v[i], part[i]);
  }
  __syncthreads();
#pragma unroll
  for (int i = 0; i < kFftPerThread; ++i) {
    const uint32_t e = tid + i * nthreads;
    if (e < total) lds[e] = v[i];
  }
  __syncthreads();
}

// Transforms every line in place.  The block's lines hold at most
// kFftPerThread * nthreads values; begins and ends with a barrier.  KIND: fft_kind
// of the plan.
template <int KIND>
__device__ inline void fft_lines(float2* lds, const float2* tw, uint32_t lines, FastDiv div_lines, const FftPlan& p,
                                 uint32_t tid, uint32_t nthreads) {
  __syncthreads();
  uint32_t ns = 1;
  for (uint32_t s = 0; s < p.passes; ++s) {
    const uint32_t r = p.radix[s];
    const FastDiv d = p.div_ns[s];
    switch (r) {
      case 8: fft_pass<8>(lds, tw, lines, div_lines, p, ns, d, tid, nthreads); break;
      case 4: fft_pass<4>(lds, tw, lines, div_lines, p, ns, d, tid, nthreads); break;
      case 2: fft_pass<2>(lds, tw, lines, div_lines, p, ns, d, tid, nthreads); break;
      default:
        if constexpr (KIND >= kFftSmooth) {
          if (r == 3) fft_pass<3>(lds, tw, lines, div_lines, p, ns, d, tid, nthreads);
          else if (r == 5) fft_pass<5>(lds, tw, lines, div_lines, p, ns, d, tid, nthreads);
          else if (r == 7) fft_pass<7>(lds, tw, lines, div_lines, p, ns, d, tid, nthreads);
          else if constexpr (KIND == kFftPrimes) fft_pass_prime(lds, tw, lines, div_lines, p, r, ns, d, tid, nthreads);
        }
        break;
    }
    ns *= r;
  }
}

}  // namespace rflbm

// Membrane force and trapezoid weights on gfx950: the step that produces the far-field
// sum's inputs on the device.
//
//   f = -kappa_b X_ssss + (sigma X_s)_s            (eq. (elastic_force))
//   w = |X_alpha| 2 pi / N                          (the ds of eq. (single_layer))
//
// Arclength derivatives are spectral (Section 2.2.1): d/ds = (1/|X_alpha|) d/dalpha with
// d/dalpha exact on the band-limited interpolant of the N points alpha_k = 2 pi k / N.
// On the grid that operator is the circulant matrix with first column
//   d_0 = 0,  d_m = (1/2) (-1)^m cot(pi m / N)  (N even),  (1/2) (-1)^m csc(pi m / N)  (N odd),
// which equals multiplying Fourier mode k by i k with the even-N Nyquist mode dropped.  The weights sum
// to zero, so the points enter it relative to the vesicle's first point: rounding then scales with the
// vesicle's extent, not with its distance from the origin.  It is applied as a direct O(N^2) product in float64
// (the fourth derivative amplifies rounding by up to (N/2)^4) on the matrix cores.
//
// The product.  Points i = 16 p + r in blocks p of 16: with j = 16 (p - t) + s,
//   (D u)_i = sum_t sum_s T_t[r][s] u_j,   T_t[r][s] = d[(r - s + 16 t) mod N],
// so the 16 x 16 matrix T_t multiplies all blocks at once: the columns of the other operand are the blocks (moved by
// t) of both components, eight blocks x two components to a 16-column accumulator.  t runs over the ceil(N / 16)
// blocks; where N is no multiple of 16 the pairs of the last t that wrap round a second time, 16 t - s > N - 16, are
// dropped.  Operands come from LDS (d and u extended by their period, so no index is reduced), two 8-byte reads for
// 64 cycles of matrix work: the matrix cores bound it.
// One wavefront holds 128 points; a vesicle of up to 128 points is one wavefront's work, a larger one (up to 1024) is
// shared by a workgroup's eight, 128 points each.
#include <hip/hip_runtime.h>
#include <math.h>
#include <stdint.h>

#include <type_traits>

#include "vesnet_internal.h"

namespace vesnet {

namespace {

constexpr int kMaxN = 1024;
constexpr int kWaves = 8;
constexpr int kB = 64 * kWaves;
constexpr int kWavePoints = 128;  // of one wavefront: eight blocks x two components are the 16 columns
constexpr int kValues = 4;        // accumulator rows of a lane

typedef double double4v __attribute__((ext_vector_type(4)));

__device__ __forceinline__ int clamp_i(int x, int lo, int hi) { return x < lo ? lo : (x > hi ? hi : x); }

// LDS doubles of a vesicle of up to `points` points: d at indices -15 .. points - 1 (one spare), then u at indices
// -(points - 16) .. points - 1.
constexpr int region_doubles(int points) { return points + 16 + 40 * (points / 8 - 1); }

// LDS position of u_j: the components side by side, eight spare doubles every sixteen points, which puts the eight
// blocks that one read touches on different banks.
__device__ __forceinline__ int upos(int j) { return 2 * j + 8 * (j >> 4); }

// The other component's value at the same point (neighbouring lanes hold x and y).
__device__ __forceinline__ double other_component(double v) {
  const int lo = __builtin_amdgcn_update_dpp(0, __double2loint(v), 0xB1, 0xF, 0xF, false);  // quad_perm 1, 0, 3, 2
  const int hi = __builtin_amdgcn_update_dpp(0, __double2hiint(v), 0xB1, 0xF, 0xF, false);
  return __hiloint2double(hi, lo);
}

// One vesicle of n points, worked on by one wavefront (kCoop = false) or by the whole workgroup.  Lane l of a
// wavefront holds component l & 1 of points 16 p + (l >> 4) + 4 q, q = 0 .. 3, of its block p.
template <bool kCoop>
struct Curve {
  double* d;  // d[-15 .. 16 nb - 1]
  double* u;  // positions of j = -(16 nb - 16) .. 16 nb - 1
  int n, nb;  // points, blocks of 16
  int p, c, k4;
  bool live;  // this wavefront has points

  __device__ __forceinline__ Curve(double* lds, int points) {
    const int lane = threadIdx.x & 63;
    const int wave = kCoop ? threadIdx.x >> 6 : 0;
    n = points;
    nb = (n + 15) >> 4;
    p = 8 * wave + ((lane & 15) >> 1);
    c = lane & 1;
    k4 = lane >> 4;
    live = 8 * wave < nb;
    d = lds + 15;
    u = lds + 16 * nb + 16 + 40 * (nb - 1);
  }

  __device__ __forceinline__ void sync() const {
    if constexpr (kCoop) __syncthreads();
    else wave_sync();
  }

  __device__ __forceinline__ int point(int q) const { return 16 * p + k4 + 4 * q; }
  __device__ __forceinline__ bool owns(int q) const { return point(q) < n; }
  __device__ __forceinline__ int at(int q) const { return min(point(q), n - 1); }  // for loads without a branch

  // Sets a[k] for k = at, at +- n, ... in [lo, 16 nb).
  template <class Put>
  __device__ __forceinline__ void periodic(int at, int lo, const Put& put) const {
    if (n >= 16) {  // lo >= 1 - n and 16 nb <= n + 15: at most one period to either side
      put(at);
      if (at - n >= lo) put(at - n);
      if (at + n < 16 * nb) put(at + n);
    } else {
      for (int k = at - 15 * n; k < 16; k += n)
        if (k >= lo) put(k);
    }
  }

  // The weights, d_{N-m} = -d_m.
  __device__ __forceinline__ void put_weight(int m, double v) const {
    periodic(m, -15, [&](int k) { d[k] = v; });
  }
  __device__ __forceinline__ void weights() const {
    const int step = kCoop ? kB : 64, at = kCoop ? threadIdx.x : threadIdx.x & 63;
    for (int m = at; 2 * m <= n; m += step) {
      double v = 0.0;
      if (m > 0 && 2 * m < n) {
        double s, co;
        sincospi((double)m / (double)n, &s, &co);
        const double sg = (m & 1) ? -0.5 : 0.5;
        v = (n & 1) ? sg / s : sg * co / s;
        put_weight(n - m, -v);
      }
      put_weight(m, v);
    }
  }

  // u for the next product (the previous one is done with it; the caller synchronises before and after).
  __device__ __forceinline__ void store(const double (&v)[kValues]) const {
#pragma unroll
    for (int q = 0; q < kValues; ++q) {
      if (owns(q)) periodic(point(q), 16 - 16 * nb, [&](int k) { u[upos(k) + c] = v[q]; });
    }
  }

  // D u at this lane's points (a lane beyond the last point repeats the last block, its values are not used).
  __device__ __forceinline__ void product(double (&out)[kValues]) const {
    double4v acc0 = {0.0, 0.0, 0.0, 0.0}, acc1 = {0.0, 0.0, 0.0, 0.0};
    if (live) {
      const double* dp = d + ((threadIdx.x & 15) - k4);
      const double* up = u + 40 * min(p, nb - 1) + 2 * k4 + c;
      double a[4], b[4];  // the operands of one t, read while the one before is multiplied
      const auto load = [&]() __attribute__((always_inline)) {
#pragma unroll
        for (int k = 0; k < 4; ++k) {
          a[k] = dp[-4 * k];
          b[k] = up[8 * k];
        }
        dp += 16;
        up -= 40;
      };
      load();
      asm volatile("; t = 0");  // keeps these reads apart from the loop's (merged, every t would copy the accumulators)
      for (int t = 0; t < nb - 1; ++t) {
        const double a0 = a[0], a1 = a[1], a2 = a[2], a3 = a[3], b0 = b[0], b1 = b[1], b2 = b[2], b3 = b[3];
        load();
        acc0 = __builtin_amdgcn_mfma_f64_16x16x4f64(a0, b0, acc0, 0, 0, 0);
        acc1 = __builtin_amdgcn_mfma_f64_16x16x4f64(a1, b1, acc1, 0, 0, 0);
        acc0 = __builtin_amdgcn_mfma_f64_16x16x4f64(a2, b2, acc0, 0, 0, 0);
        acc1 = __builtin_amdgcn_mfma_f64_16x16x4f64(a3, b3, acc1, 0, 0, 0);
      }
      const int x = 16 * nb - n;  // s < x wraps round
      acc0 = __builtin_amdgcn_mfma_f64_16x16x4f64(a[0], k4 < x ? 0.0 : b[0], acc0, 0, 0, 0);
      acc1 = __builtin_amdgcn_mfma_f64_16x16x4f64(a[1], 4 + k4 < x ? 0.0 : b[1], acc1, 0, 0, 0);
      acc0 = __builtin_amdgcn_mfma_f64_16x16x4f64(a[2], 8 + k4 < x ? 0.0 : b[2], acc0, 0, 0, 0);
      acc1 = __builtin_amdgcn_mfma_f64_16x16x4f64(a[3], 12 + k4 < x ? 0.0 : b[3], acc1, 0, 0, 0);
    }
#pragma unroll
    for (int q = 0; q < kValues; ++q) out[q] = acc0[q] + acc1[q];
  }

  __device__ __forceinline__ void derivative(const double (&v)[kValues], double (&out)[kValues]) const {
    sync();
    store(v);
    sync();
    product(out);
  }
};

// The vesicles of this workgroup: `per` consecutive ones per step of the grid.  body(curve, j0) runs with one
// wavefront for each vesicle of up to 128 points and with the whole workgroup for larger ones; too_large(j0, n)
// with the whole workgroup for those of more than 1024 points.
template <class Body, class TooLarge>
__device__ __forceinline__ void for_vesicles(double* lds, const int32_t* __restrict__ off, int M, int P, int per,
                                             const Body& body, const TooLarge& too_large) {
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  for (int v0 = blockIdx.x * per; v0 < M; v0 += gridDim.x * per) {
    const int v1 = min(v0 + per, M);
    if (v0 + wave < v1) {
      const int j0 = clamp_i(off[v0 + wave], 0, P);
      const int n = max(j0, clamp_i(off[v0 + wave + 1], 0, P)) - j0;
      if (n > 0 && n <= kWavePoints)
        body(Curve<false>(lds + wave * region_doubles(kWavePoints), n), j0);
    }
    for (int v = v0; v < v1; ++v) {
      const int j0 = clamp_i(off[v], 0, P);
      const int n = max(j0, clamp_i(off[v + 1], 0, P)) - j0;
      if (n <= kWavePoints) continue;
      if (n > kMaxN) {
        too_large(j0, n);
        continue;
      }
      __syncthreads();  // the wavefronts' own vesicles are done with LDS
      body(Curve<true>(lds, n), j0);
      __syncthreads();
    }
  }
}

constexpr int kLdsDoubles = kWaves * region_doubles(kWavePoints) > region_doubles(kMaxN)
                                ? kWaves * region_doubles(kWavePoints) : region_doubles(kMaxN);

// Five products of 32 matrix instructions (64 cycles each) at 128 points: 2000 x 128 is two wavefronts on every SIMD
// and 8.5 us of matrix work; 49.9 -> 18.8 us (before: vector FMAs, whose operands came from LDS at three reads for four
// FMAs, and a second launch for vesicles above the wavefront form).
__global__ __launch_bounds__(kB) void k_elastic(const double* __restrict__ X, const double* __restrict__ sigma,
                                                double kappa_b, const int32_t* __restrict__ off, int M, int P, int per,
                                                double* __restrict__ f, double* __restrict__ w) {
  __shared__ double lds[kLdsDoubles];
  const auto one = [&](const auto& cv, int j0) __attribute__((always_inline)) {
    const int n = cv.n;
    const double* Xc = X + (cv.c ? P : 0) + j0;
    double* fc = f + (cv.c ? P : 0) + j0;
    double sg[kValues], a[kValues], jinv[kValues], tension[kValues];
    const double* sg0 = sigma ? sigma + j0 : Xc;  // not used without tension
    const double x0 = Xc[0];
#pragma unroll
    for (int q = 0; q < kValues; ++q) {
      a[q] = Xc[cv.at(q)] - x0;
      sg[q] = sg0[cv.at(q)];
      tension[q] = 0.0;
    }
    cv.weights();
    cv.derivative(a, a);  // X_alpha
#pragma unroll
    for (int q = 0; q < kValues; ++q) {
      const double o = other_component(a[q]);
      const double J = sqrt(a[q] * a[q] + o * o);
      jinv[q] = 1.0 / J;
      if (cv.c == 0 && cv.owns(q)) w[j0 + cv.point(q)] = J * (6.28318530717958647693 / (double)n);
      a[q] *= jinv[q];  // X_s
      sg[q] *= a[q];
    }
    if (sigma) {  // (sigma X_s)_s
      cv.derivative(sg, tension);
#pragma unroll
      for (int q = 0; q < kValues; ++q) tension[q] *= jinv[q];
    }
    for (int pass = 0; pass < 3; ++pass) {  // X_ss, X_sss, X_ssss
      cv.derivative(a, a);
#pragma unroll
      for (int q = 0; q < kValues; ++q) a[q] *= jinv[q];
    }
#pragma unroll
    for (int q = 0; q < kValues; ++q)
      if (cv.owns(q)) fc[cv.point(q)] = fma(-kappa_b, a[q], tension[q]);
  };
  const auto too_large = [&](int j0, int n) {
    for (int i = threadIdx.x; i < n; i += kB) {
      f[j0 + i] = NAN;
      f[P + j0 + i] = NAN;
      w[j0 + i] = NAN;
    }
  };
  for_vesicles(lds, off, M, P, per, one, too_large);
}

// CreateNearLayers (Algorithm 4, Section 3.3): node a = l * n + k of vesicle v is membrane point
// k moved along the outward unit normal by d_l = (l - 2) h_v / 2, l = 0..4.  The tangent is the
// spectral X_alpha / |X_alpha|; the outward side is fixed by the sign of the enclosed signed area
// (trapezoid rule of (x y_alpha - y x_alpha) / 2), so either orientation of the points works.
// One product of the force's kind; 100 B per point.  2000 x 32: 10.2 -> 8.5 us; 2000 x 128: 20.6 -> 15.0 us.
__global__ __launch_bounds__(kB) void k_near_layers(const double* __restrict__ X, const double* __restrict__ w,
                                                    const int32_t* __restrict__ off, int M, int P, int per,
                                                    double* __restrict__ layers) {
  __shared__ double lds[kLdsDoubles];
  __shared__ double red[kWaves];
  const size_t P5 = (size_t)5 * P;
  const auto undefined = [&](int j0, int n, int at, int step) {
    for (int a = at; a < 5 * n; a += step) {
      layers[(size_t)5 * j0 + a] = NAN;
      layers[P5 + (size_t)5 * j0 + a] = NAN;
    }
  };
  const auto one = [&](const auto& cv, int j0) __attribute__((always_inline)) {
    const int n = cv.n;
    if (n < 3) {
      undefined(j0, n, threadIdx.x & 63, 64);
      return;
    }
    const double* Xc = X + (cv.c ? P : 0) + j0;
    double* lc = layers + (cv.c ? P5 : 0) + (size_t)5 * j0;
    double x[kValues], u[kValues], a[kValues];
    const double x0 = Xc[0];
#pragma unroll
    for (int q = 0; q < kValues; ++q) {
      x[q] = Xc[cv.at(q)];
      u[q] = x[q] - x0;
    }
    const double h = wave_mean_spacing(w + j0, n);
    cv.weights();
    cv.derivative(u, a);  // X_alpha
    double part = 0.0;
#pragma unroll
    for (int q = 0; q < kValues; ++q) {
      const double o = other_component(a[q]);
      const double jinv = 1.0 / sqrt(a[q] * a[q] + o * o);
      if (cv.owns(q)) part += cv.c ? -(u[q] * o) : u[q] * o;
      a[q] = cv.c ? -o * jinv : o * jinv;  // tangent turned clockwise: outward when counter-clockwise
    }
#pragma unroll
    for (int m = 32; m >= 1; m >>= 1) part += __shfl_xor(part, m, 64);
    if constexpr (!std::is_same_v<std::decay_t<decltype(cv)>, Curve<false>>) {
      if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = part;
      __syncthreads();
      part = 0.0;
#pragma unroll
      for (int k = 0; k < kWaves; ++k) part += red[k];
    }
    const double orient = part >= 0.0 ? 1.0 : -1.0;
#pragma unroll
    for (int q = 0; q < kValues; ++q) {
      if (!cv.owns(q)) continue;
#pragma unroll
      for (int l = 0; l < 5; ++l) lc[l * n + cv.point(q)] = fma(0.5 * (double)(l - 2) * h, orient * a[q], x[q]);
    }
  };
  for_vesicles(lds, off, M, P, per, one, [&](int j0, int n) { undefined(j0, n, threadIdx.x, kB); });
}

// Vesicles per workgroup.  While there are fewer workgroups than compute units each gets a vesicle of its own (two
// wavefronts on one SIMD share its matrix core: 13.9 us for 1024 x 128, 21.6 us for 2000); beyond, up to eight share
// one, a wavefront each.  Vesicles above 128 points on average take a workgroup each, since one after the other they
// would leave most of the chip idle (200 x 200: 16.7 us, before 46.3 us with a wavefront each; 64 x 1024: 546 -> 96 us).
int vesicles_per_block(int M, int P) {
  if ((int64_t)P > (int64_t)kWavePoints * M) return 1;
  const int per = (M + 255) / 256;
  return per < kWaves ? per : kWaves;
}

int blocks(int M, int per) {
  const int g = (M + per - 1) / per;
  return g < 65535 ? g : 65535;
}

}  // namespace

hipError_t launch_near_layers(const double* X, const double* w, const int32_t* off, int M, int P, double* layers,
                              void* stream) {
  if (M == 0 || P == 0) return hipSuccess;
  const int per = vesicles_per_block(M, P);
  hipLaunchKernelGGL(k_near_layers, dim3(blocks(M, per)), dim3(kB), 0, reinterpret_cast<hipStream_t>(stream), X, w, off,
                     M, P, per, layers);
  return hipGetLastError();
}

hipError_t launch_elastic(const double* X, const double* sigma, double kappa_b, const int32_t* off, int M, int P,
                          double* f, double* w, void* stream) {
  if (M == 0 || P == 0) return hipSuccess;
  const int per = vesicles_per_block(M, P);
  hipLaunchKernelGGL(k_elastic, dim3(blocks(M, per)), dim3(kB), 0, reinterpret_cast<hipStream_t>(stream), X, sigma,
                     kappa_b, off, M, P, per, f, w);
  return hipGetLastError();
}

}  // namespace vesnet

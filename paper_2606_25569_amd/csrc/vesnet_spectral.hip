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
// shared by a workgroup's, 128 points each.  Many vesicles of 129 to 256 points on average take workgroups of two
// wavefronts, and a second launch does the larger ones.  Many vesicles of few points, whose 16 x 16 blocks would be mostly
// padding, take their force by vector instructions instead (k_elastic_small).
#include <hip/hip_runtime.h>
#include <math.h>
#include <stdint.h>

#include <type_traits>

#include "vesnet_internal.h"

namespace vesnet {

namespace {

constexpr int kMaxN = 1024;
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

// One vesicle of n points, worked on by kW wavefronts, all of the workgroup's if more than one.  Lane l of a
// wavefront holds component l & 1 of points 16 p + (l >> 4) + 4 q, q = 0 .. 3, of its block p.
template <int kW>
struct Curve {
  static constexpr bool kCoop = kW > 1;
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
      for (int k = at - (at - lo) / n * n; k < 16; k += n) put(k);
    }
  }

  // The weights, d_{N-m} = -d_m.
  __device__ __forceinline__ void put_weight(int m, double v) const {
    periodic(m, -15, [&](int k) { d[k] = v; });
  }
  __device__ __forceinline__ void weights() const {
    const int step = 64 * kW, at = kCoop ? threadIdx.x : threadIdx.x & 63;
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

// LDS doubles of a workgroup of kW wavefronts that takes vesicles of up to kCap points.
template <int kW, int kCap>
constexpr int lds_doubles() {
  return kW * region_doubles(kWavePoints) > region_doubles(kCap) ? kW * region_doubles(kWavePoints) : region_doubles(kCap);
}

// The vesicles of more than min_n and up to kCap points.  body(curve, j0) runs with one wavefront for each of up to 128
// points, `per` consecutive ones to a workgroup, and with the whole workgroup for larger ones, which are dealt to the
// workgroups in turn, each turn moved on by one, so that neither neighbours nor every second one meet in the same (200
// neighbours of 200 points among 2200: 105 -> 24 us).  too_large(j0, n) with the whole workgroup for those of more than
// 1024 points, where kCap is 1024.
template <int kW, int kCap, class Body, class TooLarge>
__device__ __forceinline__ void for_vesicles(double* lds, const int32_t* __restrict__ off, int M, int P, int per,
                                             int min_n, const Body& body, const TooLarge& too_large) {
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
  const auto points = [&](int a, int b, int& j0) {
    j0 = clamp_i(a, 0, P);
    return max(j0, clamp_i(b, 0, P)) - j0;
  };
  const auto dealt = [&](int turn) {  // this workgroup's vesicle of that turn, M for none (turns are fewer than workgroups)
    const int at = blockIdx.x + turn, grid = gridDim.x;
    const int64_t v = (int64_t)turn * grid + (at < grid ? at : at - grid);
    return v < M ? (int)v : M;
  };
  int j0;
  // the sizes of the first 64 turns' vesicles are on their way while the wavefronts' own are worked on
  int v = dealt(lane);
  int a = off[min(v, M - 1)], b = off[min(v, M - 1) + 1];
  for (int v0 = blockIdx.x * per; v0 < M; v0 += gridDim.x * per) {
    if (wave < per && v0 + wave < M) {
      const int n = points(off[v0 + wave], off[v0 + wave + 1], j0);
      if (n > min_n && n <= kWavePoints) body(Curve<1>(lds + wave * region_doubles(kWavePoints), n), j0);
    }
  }
  for (int turn0 = 0;;) {
    const int n0 = v < M ? points(a, b, j0) : 0;
    for (unsigned long long todo = __ballot(n0 > kWavePoints && n0 > min_n); todo; todo &= todo - 1) {
      const int u = dealt(turn0 + __ffsll(todo) - 1);
      const int n = points(off[u], off[u + 1], j0);
      if (n > kCap) {
        if (kCap == kMaxN) too_large(j0, n);
        continue;
      }
      __syncthreads();  // LDS is free
      body(Curve<kW>(lds, n), j0);
    }
    turn0 += 64;
    if ((int64_t)turn0 * gridDim.x >= M) break;
    v = dealt(turn0 + lane);
    a = off[min(v, M - 1)];
    b = off[min(v, M - 1) + 1];
  }
}

// Five products of 32 matrix instructions (64 cycles each) at 128 points: 2000 x 128 is two wavefronts on every SIMD
// and 8.5 us of matrix work; 49.9 -> 18.8 us (before: vector FMAs, whose operands came from LDS at three reads for four
// FMAs, and a second launch for vesicles above the wavefront form).
template <int kW, int kCap>
__global__ __launch_bounds__(64 * kW) void k_elastic(const double* __restrict__ X, const double* __restrict__ sigma,
                                                     double kappa_b, const int32_t* __restrict__ off, int M, int P, int per,
                                                     int min_n, double* __restrict__ f, double* __restrict__ w) {
  __shared__ double lds[lds_doubles<kW, kCap>()];
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
    for (int i = threadIdx.x; i < n; i += 64 * kW) {
      f[j0 + i] = NAN;
      f[P + j0 + i] = NAN;
      w[j0 + i] = NAN;
    }
  };
  for_vesicles<kW, kCap>(lds, off, M, P, per, min_n, one, too_large);
}

// The force of vesicles of up to 64 points by vector instructions, a wavefront each, lane i owning point i: u is stored
// twice (u2[j] = u2[j + n] = u_j), (D u)_i = sum_m d_m u2[i + n - m].  Its few registers and 1.5 KB of LDS let 32 wavefronts
// share a compute unit, where the matrix form has 12 and pads every vesicle to blocks of 16 points: 10,000 vesicles of 8
// points 15 us against 34, of 24 points 24 against 40.
constexpr int kSmallN = 64;

__global__ __launch_bounds__(64) void k_elastic_small(const double* __restrict__ X, const double* __restrict__ sigma,
                                                      double kappa_b, const int32_t* __restrict__ off, int M, int P,
                                                      double* __restrict__ f, double* __restrict__ w) {
  __shared__ double d[kSmallN];
  __shared__ double2 u2[2 * kSmallN];
  const int i = threadIdx.x;
  for (int v = blockIdx.x; v < M; v += gridDim.x) {
    const int j0 = clamp_i(off[v], 0, P);
    const int n = max(j0, clamp_i(off[v + 1], 0, P)) - j0;
    if (n == 0 || n > kSmallN) continue;
    const bool live = i < n;
    const int j = j0 + (live ? i : 0);
    const double sg = sigma ? sigma[j] : 0.0;
    const auto product = [&](double2 u) {
      wave_sync();  // the previous product is done
      if (live) u2[i] = u2[i + n] = u;
      wave_sync();
      double2 s = make_double2(0.0, 0.0);
      if (live)
        for (int m = 0; m < n; ++m) {  // d_0 = 0 too: it carries a value that is not finite
          const double2 t = u2[i + n - m];
          s.x = fma(d[m], t.x, s.x);
          s.y = fma(d[m], t.y, s.y);
        }
      return s;
    };
    wave_sync();  // the previous vesicle is done with d
    if (live) {
      double c = 0.0;
      if (i > 0) {
        double s, co;
        sincospi((double)i / (double)n, &s, &co);
        const double sign = (i & 1) ? -0.5 : 0.5;
        c = (n & 1) ? sign / s : sign * co / s;
      }
      d[i] = c;
    }
    double2 a = product(make_double2(X[j] - X[j0], X[P + j] - X[P + j0]));  // X_alpha
    const double J = sqrt(a.x * a.x + a.y * a.y), jinv = 1.0 / J;
    if (live) w[j] = J * (6.28318530717958647693 / (double)n);
    a = make_double2(a.x * jinv, a.y * jinv);  // X_s
    double2 t = make_double2(0.0, 0.0);
    if (sigma) {  // (sigma X_s)_s
      t = product(make_double2(sg * a.x, sg * a.y));
      t = make_double2(t.x * jinv, t.y * jinv);
    }
    for (int pass = 0; pass < 3; ++pass) {  // X_ss, X_sss, X_ssss
      a = product(a);
      a = make_double2(a.x * jinv, a.y * jinv);
    }
    if (live) {
      f[j] = fma(-kappa_b, a.x, t.x);
      f[P + j] = fma(-kappa_b, a.y, t.y);
    }
  }
}

// CreateNearLayers (Algorithm 4, Section 3.3): node a = l * n + k of vesicle v is membrane point
// k moved along the outward unit normal by d_l = (l - 2) h_v / 2, l = 0..4.  The tangent is the
// spectral X_alpha / |X_alpha|; the outward side is fixed by the sign of the enclosed signed area
// (trapezoid rule of (x y_alpha - y x_alpha) / 2), so either orientation of the points works.
// One product of the force's kind; 100 B per point.  2000 x 32: 10.2 -> 8.5 us; 2000 x 128: 20.6 -> 15.0 us.
template <int kW, int kCap>
__global__ __launch_bounds__(64 * kW) void k_near_layers(const double* __restrict__ X, const double* __restrict__ w,
                                                         const int32_t* __restrict__ off, int M, int P, int per,
                                                         int min_n, double* __restrict__ layers) {
  __shared__ double lds[lds_doubles<kW, kCap>()];
  __shared__ double red[kW];
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
    if constexpr (std::decay_t<decltype(cv)>::kCoop) {
      if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = part;
      __syncthreads();
      part = 0.0;
#pragma unroll
      for (int k = 0; k < kW; ++k) part += red[k];
    }
    const double orient = part >= 0.0 ? 1.0 : -1.0;
#pragma unroll
    for (int q = 0; q < kValues; ++q) {
      if (!cv.owns(q)) continue;
#pragma unroll
      for (int l = 0; l < 5; ++l) lc[l * n + cv.point(q)] = fma(0.5 * (double)(l - 2) * h, orient * a[q], x[q]);
    }
  };
  for_vesicles<kW, kCap>(lds, off, M, P, per, min_n, one, [&](int j0, int n) { undefined(j0, n, threadIdx.x, 64 * kW); });
}

// Vesicles per workgroup of the matrix form.  While there are fewer workgroups than compute units each gets a vesicle of
// its own (two wavefronts on one SIMD share its matrix core: 13.9 us for 1024 x 128, 21.6 us for 2000); beyond, up to
// eight share one, a wavefront each.  Vesicles above 128 points on average take a workgroup each, since one after the
// other they would leave most of the chip idle (200 x 200: 16.7 us, before 46.3 us with a wavefront each; 64 x 1024: 546
// -> 96 us).
int vesicles_per_block(int M, int P) {
  if ((int64_t)P > (int64_t)kWavePoints * M) return 1;
  const int per = (M + 255) / 256;
  return per < 8 ? per : 8;
}

int blocks(int M, int per) {
  const int g = (M + per - 1) / per;
  return g < 65535 ? g : 65535;
}

// launch(wavefronts, cap, grid, per, min_n) of the matrix form for the vesicles of more than done points, once, or twice
// for more than `many` vesicles of 129 to 256 points on average: workgroups of two wavefronts with LDS for 256 points, of
// which six fit where one of eight does, six of them idle, then the larger ones.  2000 vesicles of 160 points: force 91 ->
// 64 us, layers 47 -> 28.  (A grid is no smaller than the turns in which it deals them: 8, or M / 65535.)
template <class Launch>
void launch_matrix(int M, int P, int many, int done, const Launch& launch) {
  constexpr std::integral_constant<int, 8> eight{};
  constexpr std::integral_constant<int, kMaxN> all{};
  if (M > many && P > kWavePoints * (int64_t)M && P <= 256 * (int64_t)M) {
    launch(std::integral_constant<int, 2>{}, std::integral_constant<int, 256>{}, blocks(M, 1), 1, done);
    launch(eight, all, M < 512 ? M : 512 + M / 512, 1, 256);
  } else {
    const int per = done > 0 ? 8 : vesicles_per_block(M, P);
    launch(eight, all, blocks(M, per), per, done);
  }
}

}  // namespace

hipError_t launch_near_layers(const double* X, const double* w, const int32_t* off, int M, int P, double* layers,
                              void* stream) {
  if (M == 0 || P == 0) return hipSuccess;
  launch_matrix(M, P, 512, 0, [&](auto kW, auto kCap, int grid, int per, int min_n) {
    hipLaunchKernelGGL((k_near_layers<kW.value, kCap.value>), dim3(grid), dim3(64 * kW.value), 0,
                       reinterpret_cast<hipStream_t>(stream), X, w, off, M, P, per, min_n, layers);
  });
  return hipGetLastError();
}

hipError_t launch_elastic(const double* X, const double* sigma, double kappa_b, const int32_t* off, int M, int P,
                          double* f, double* w, void* stream) {
  if (M == 0 || P == 0) return hipSuccess;
  hipStream_t st = reinterpret_cast<hipStream_t>(stream);
  // more than the matrix form holds at once, and small: 2,500 vesicles of 24 points 12.5 us against 17.0; 2,000 of 16,
  // one round of the matrix form, take 9.4 there
  int done = 0;
  if (M > 2048 && P <= 24 * (int64_t)M) {
    done = kSmallN;
    hipLaunchKernelGGL(k_elastic_small, dim3(blocks(M, 1)), dim3(64), 0, st, X, sigma, kappa_b, off, M, P, f, w);
  }
  launch_matrix(M, P, 1024, done, [&](auto kW, auto kCap, int grid, int per, int min_n) {
    hipLaunchKernelGGL((k_elastic<kW.value, kCap.value>), dim3(grid), dim3(64 * kW.value), 0, st, X, sigma, kappa_b, off,
                       M, P, per, min_n, f, w);
  });
  return hipGetLastError();
}

}  // namespace vesnet

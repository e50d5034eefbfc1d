// Near-field interpolation on gfx950 (Section 3.3, Algorithm 4 interpolateInNearField).
//
// Each vesicle v carries n = 5 N_v nodes x_a (its five layers) with known velocities u_a.  The
// Gaussian radial basis interpolant  s(x) = sum_a phi(|x - x_a|) c_a,  phi(r) = exp(-r^2 / (eps h_v)^2),
// takes its coefficients from the symmetric positive definite system K c = u, K_ab = phi(|x_a - x_b|),
// which the paper solves by batched Cholesky factorisation.
//
// k_rbf_fit: one wavefront per vesicle factors K = L L^T in float64 by a left-looking blocked
// algorithm on 32 x 32 tiles, in an order that keeps the nodes of one membrane point together (node b = 5 k + l is
// layer l of point k): entries of points far apart along the curve are below 1e-19 of the diagonal, so the factor of
// a long vesicle is nearly banded.  Tile (I, J) is zero left of the first tile column f(I) whose bounding box comes
// within that distance of tile row I's (a Cholesky factor keeps the envelope of its matrix), and no work is done
// there: 20 x 20 tiles of a 128-point vesicle hold about 70 of 210 lower tiles, and a seventh of the products.  The
// entries of K are recomputed from the node coordinates when a panel needs them, so only L is stored (in a
// per-wavefront slot of the tile workspace, lower tiles packed).  Every stored tile is in the layout of a matrix
// instruction's operand, so the products load it from the slot straight into registers, each lane what it stored
// itself (no LDS staging, no barrier); the finished products pass through LDS once to change layout.
// Each diagonal tile is factored and inverted, W = L_JJ^{-1}, by 16 x 16 blocks with one row per lane (values of a
// pivot row come by DPP row broadcasts), the rest on the matrix cores; W replaces L_JJ in the slot (no later panel
// reads L_JJ) and L_IJ = T_IJ W^T.  The two right-hand sides are carried through the panels, y_J = W (u_J - sum_k
// L_Jk y_k), and the back substitution L^T c = y takes c_J = W_JJ^T (y_J - sum_{I>J} L_IJ^T c_I).  The rows are padded
// to a multiple of 32 with an identity block, which leaves the factor and the solution unchanged.
// What bounds it: at 2000 x 32, two wavefronts per SIMD, issue (19,375 VALU instructions and 736 FP64 matrix
// instructions each, about 45% and 24% of the time) and what of the serial pivots' latency the other wavefront leaves
// uncovered; a fifth less tile traffic changed nothing.  With fewer or longer vesicles it is the latency of a panel,
// about 40 us at 128 points.  2000 x 32: 294 -> 171 us; 48 x 32:
// 149 -> 82 us; 500 x 128: 4.22 -> 0.72 ms; 200 x 200: 13.6 -> 1.31 ms (before: layer-major order, every lower tile,
// row-major tiles staged through LDS, 32-row pivots by lane reads).
//
// k_rbf_eval_near: one wavefront per near (target, vesicle) pair sums phi c over the vesicle's nodes
// and adds the result into the target's velocity.
#include <hip/hip_runtime.h>
#include <math.h>
#include <stdint.h>

#include <type_traits>
#include <utility>

#include "vesnet_internal.h"

namespace vesnet {

namespace {

constexpr int kT = 32;           // tile edge
constexpr int kLd = kT + 1;      // LDS row stride in doubles (conflict-free column reads)
constexpr int kFW = 64;          // one wavefront per vesicle
constexpr int kMaxNodes = 1000;  // 5 x 200 points: 32 tile rows, one lane each for the envelope

__device__ __forceinline__ int clamp_i(int x, int lo, int hi) { return x < lo ? lo : (x > hi ? hi : x); }

// Packed lower tiles: tile (I, J), J <= I, at index I (I + 1) / 2 + J.
__device__ __forceinline__ size_t tile_index(int I, int J) { return (size_t)I * (I + 1) / 2 + J; }

// A tile in operand layout: lane i + 16 k of the wavefront holds elements (16 R + i, 4 s + k), R = 0, 1, s = 0 .. 7:
// the A operand of a product with the tile on the left, and the B operand of one with its transpose on the right.
// In the slot each lane's elements are pairs (s, s + 1) at double2 index (4 R + s / 2) 64 + lane.
typedef double double4v __attribute__((ext_vector_type(4)));

struct Tile {
  double e[2][8];
};

__device__ __forceinline__ Tile load_tile(const double2* __restrict__ t, int lane) {
  Tile r;
#pragma unroll
  for (int R = 0; R < 2; ++R)
#pragma unroll
    for (int s = 0; s < 4; ++s) {
      const double2 v = t[(4 * R + s) * kFW + lane];
      r.e[R][2 * s] = v.x;
      r.e[R][2 * s + 1] = v.y;
    }
  return r;
}

__device__ __forceinline__ void store_tile(double2* __restrict__ t, int lane, const Tile& r) {
#pragma unroll
  for (int R = 0; R < 2; ++R)
#pragma unroll
    for (int s = 0; s < 4; ++s) t[(4 * R + s) * kFW + lane] = make_double2(r.e[R][2 * s], r.e[R][2 * s + 1]);
}

// The tile in LDS (row stride kLd) in operand layout.
__device__ __forceinline__ Tile tile_from_lds(const double* __restrict__ A, int lane) {
  const int i = lane & 15, k = lane >> 4;
  Tile r;
#pragma unroll
  for (int R = 0; R < 2; ++R)
#pragma unroll
    for (int s = 0; s < 8; ++s) r.e[R][s] = A[(16 * R + i) * kLd + 4 * s + k];
  return r;
}

// Accumulators of a 32 x 32 product as four 16 x 16 blocks (R, C): lane l holds column 16 C + (l & 15) and rows
// 16 R + (l >> 4) + 4 q, q = 0..3.
typedef double4v Acc[2][2];
__device__ __forceinline__ int acc_row(int lane, int R, int q) { return R * 16 + (lane >> 4) + 4 * q; }
__device__ __forceinline__ int acc_col(int lane, int C) { return C * 16 + (lane & 15); }

// acc += a b^T; kLower: block (0, 1) left out.
template <bool kLower>
__device__ __forceinline__ void tile_gemm(Acc& acc, const Tile& a, const Tile& b) {
#pragma unroll
  for (int s = 0; s < 8; ++s) {
    acc[0][0] = __builtin_amdgcn_mfma_f64_16x16x4f64(a.e[0][s], b.e[0][s], acc[0][0], 0, 0, 0);
    acc[1][0] = __builtin_amdgcn_mfma_f64_16x16x4f64(a.e[1][s], b.e[0][s], acc[1][0], 0, 0, 0);
    acc[1][1] = __builtin_amdgcn_mfma_f64_16x16x4f64(a.e[1][s], b.e[1][s], acc[1][1], 0, 0, 0);
    if (!kLower) acc[0][1] = __builtin_amdgcn_mfma_f64_16x16x4f64(a.e[0][s], b.e[1][s], acc[0][1], 0, 0, 0);
  }
}

struct NodeView {
  const double* x;  // node coordinates of this vesicle
  const double* y;
  int n;             // nodes
  int npts;          // membrane points
  double inv_w2;     // 1 / (eps h)^2
};

// Index of node b = 5 k + l (layer l of point k) in the layer-major arrays.
__device__ __forceinline__ int node_index(int b, int npts) {
  const int k = (b * 52429) >> 18;  // b / 5 for b < 43690
  return (b - 5 * k) * npts + k;
}

// acc = -K(I, J), identity in the padding; kLower: block (0, 1) is not formed.
template <bool kLower>
__device__ __forceinline__ void minus_entries(Acc& acc, const NodeView& nv, int I, int J, int lane) {
  double xr[2][4], yr[2][4], xc[2], yc[2];
#pragma unroll
  for (int R = 0; R < 2; ++R)
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int a = node_index(min(I * kT + acc_row(lane, R, q), nv.n - 1), nv.npts);
      xr[R][q] = nv.x[a];
      yr[R][q] = nv.y[a];
    }
#pragma unroll
  for (int C = 0; C < 2; ++C) {
    const int a = node_index(min(J * kT + acc_col(lane, C), nv.n - 1), nv.npts);
    xc[C] = nv.x[a];
    yc[C] = nv.y[a];
  }
#pragma unroll
  for (int R = 0; R < 2; ++R)
#pragma unroll
    for (int C = 0; C < 2; ++C)
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int row = I * kT + acc_row(lane, R, q), col = J * kT + acc_col(lane, C);
        double e = 0.0;
        if (!(kLower && R == 0 && C == 1)) {
          const double dx = xr[R][q] - xc[C], dy = yr[R][q] - yc[C];
          e = exp(-(dx * dx + dy * dy) * nv.inv_w2);
          if (row >= nv.n || col >= nv.n) e = row == col ? 1.0 : 0.0;
        }
        acc[R][C][q] = -e;
      }
}

// -acc into LDS (row stride kLd); kLower: block (0, 1) is left alone.
template <bool kLower>
__device__ __forceinline__ void minus_to_lds(double* __restrict__ A, const Acc& acc, int lane) {
#pragma unroll
  for (int R = 0; R < 2; ++R)
#pragma unroll
    for (int C = 0; C < 2; ++C)
      if (!(kLower && R == 0 && C == 1))
#pragma unroll
        for (int q = 0; q < 4; ++q) A[acc_row(lane, R, q) * kLd + acc_col(lane, C)] = -acc[R][C][q];
}

// f(integral_constant<int, i>) for i = 0 .. N - 1, unrolled (DPP controls are immediates).
template <class F, int... I>
__device__ __forceinline__ void static_for_seq(F&& f, std::integer_sequence<int, I...>) {
  (f(std::integral_constant<int, I>{}), ...);
}
template <int N, class F>
__device__ __forceinline__ void static_for(F&& f) {
  static_for_seq(f, std::make_integer_sequence<int, N>{});
}

// The value of lane J of each row of 16 lanes, in all of its lanes.
template <int J>
__device__ __forceinline__ double row_bcast(double x) {
  long long b = __double_as_longlong(x);
  b = __builtin_amdgcn_update_dpp(b, b, 0x150 + J, 0xF, 0xF, true);
  return __longlong_as_double(b);
}

// x from lane (p + N) mod 16 of the same row of 16 lanes.
template <int N>
__device__ __forceinline__ double row_rot(double x) {
  const unsigned long long b = __builtin_bit_cast(unsigned long long, x);
  const int lo = __builtin_amdgcn_update_dpp(0, (int)(unsigned)b, 0x120 + N, 0xF, 0xF, true);
  const int hi = __builtin_amdgcn_update_dpp(0, (int)(unsigned)(b >> 32), 0x120 + N, 0xF, 0xF, true);
  return __builtin_bit_cast(double, ((unsigned long long)(unsigned)hi << 32) | (unsigned)lo);
}
// Sum over the row of 16 lanes, in all of its lanes.
__device__ __forceinline__ double row_sum(double x) {
  x += row_rot<8>(x);
  x += row_rot<4>(x);
  x += row_rot<2>(x);
  return x + row_rot<1>(x);
}

// Cholesky of a 16 x 16 block and the inverse of its factor, row i = lane & 15 of the block in this lane (every row
// of 16 lanes does the same).  Column j of the factor takes s_i = T[i][j] - sum_{m<j} L[i][m] L[j][m],
// L[j][j] = sqrt(s_j), L[i][j] = s_i / L[j][j]; column i of the inverse, W[j][i] = (delta_ij - sum_{m<j} L[j][m]
// W[m][i]) / L[j][j], takes the same broadcast values L[j][m] in the same step (held from one to the other they took
// 240 registers).  On return row holds L's row (zeros right of the diagonal) and wc W's column.
__device__ __forceinline__ void chol_inv16(double (&row)[16], double (&wc)[16], int i) {
  static_for<16>([&](auto jc) {
    constexpr int j = decltype(jc)::value;
    double sj = row[j], t = i == j ? 1.0 : 0.0;
    static_for<j>([&](auto mc) {
      constexpr int m = decltype(mc)::value;
      const double l = row_bcast<j>(row[m]);
      sj = fma(-row[m], l, sj);
      t = fma(-l, wc[m], t);
    });
    const double s2 = row_bcast<j>(sj);
    double di = __builtin_amdgcn_rsq(s2);  // 1 / sqrt(s2), refined by two Newton steps
    di = fma(0.5 * di, fma(-s2 * di, di, 1.0), di);
    di = fma(0.5 * di, fma(-s2 * di, di, 1.0), di);
    row[j] = i > j ? sj * di : (i == j ? s2 * di : 0.0);
    wc[j] = t * di;
    asm volatile("" : "+v"(wc[j]));  // here: sunk to W's stores, the inverse would need every broadcast kept (spills)
  });
}

// W = L^{-1} of the Cholesky factor of the tile in A (lower part; overwritten), into B (with zeros above the
// diagonal blocks' own).  Both in LDS, row stride kLd.
__device__ __forceinline__ void factor_invert(double* __restrict__ A, double* __restrict__ B, int lane) {
  const int i16 = lane & 15, k4 = lane >> 4;
  double row[16], wc[16];
#pragma unroll
  for (int c = 0; c < 16; ++c) row[c] = A[i16 * kLd + c];
  chol_inv16(row, wc, i16);
  if (k4 == 0) {
#pragma unroll
    for (int r = 0; r < 16; ++r) B[r * kLd + i16] = wc[r];  // W11
  } else if (k4 == 1) {
#pragma unroll
    for (int r = 0; r < 16; ++r) B[r * kLd + 16 + i16] = 0.0;  // W12
  }
  wave_sync();
  double4v l21 = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
  for (int s = 0; s < 4; ++s)  // L21 = T21 W11^T
    l21 = __builtin_amdgcn_mfma_f64_16x16x4f64(A[(16 + i16) * kLd + 4 * s + k4], B[i16 * kLd + 4 * s + k4], l21, 0, 0, 0);
  wave_sync();
#pragma unroll
  for (int q = 0; q < 4; ++q) A[(16 + k4 + 4 * q) * kLd + i16] = l21[q];
  wave_sync();
  double lo[4];  // L21 in operand layout
  double4v t22;
#pragma unroll
  for (int s = 0; s < 4; ++s) {
    lo[s] = A[(16 + i16) * kLd + 4 * s + k4];
    t22[s] = A[(16 + k4 + 4 * s) * kLd + 16 + i16];
  }
#pragma unroll
  for (int s = 0; s < 4; ++s)  // T22 - L21 L21^T
    t22 = __builtin_amdgcn_mfma_f64_16x16x4f64(-lo[s], lo[s], t22, 0, 0, 0);
  wave_sync();
#pragma unroll
  for (int q = 0; q < 4; ++q) A[(16 + k4 + 4 * q) * kLd + 16 + i16] = t22[q];
  wave_sync();
#pragma unroll
  for (int c = 0; c < 16; ++c) row[c] = A[(16 + i16) * kLd + 16 + c];
  chol_inv16(row, wc, i16);
  if (k4 == 0) {
#pragma unroll
    for (int r = 0; r < 16; ++r) B[(16 + r) * kLd + 16 + i16] = wc[r];  // W22
  }
  wave_sync();
  double4v x = {0.0, 0.0, 0.0, 0.0}, w21 = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
  for (int s = 0; s < 4; ++s)  // X = L21 W11
    x = __builtin_amdgcn_mfma_f64_16x16x4f64(lo[s], B[(4 * s + k4) * kLd + i16], x, 0, 0, 0);
#pragma unroll
  for (int s = 0; s < 4; ++s)  // W21 = -W22 X: X's accumulators are in the B operand's layout already
    w21 = __builtin_amdgcn_mfma_f64_16x16x4f64(-B[(16 + i16) * kLd + 16 + 4 * s + k4], x[s], w21, 0, 0, 0);
#pragma unroll
  for (int q = 0; q < 4; ++q) B[(16 + k4 + 4 * q) * kLd + i16] = w21[q];
  wave_sync();
}

// Entries beyond this exponent (2.9e-20) are taken as zero where a whole tile is.
constexpr double kZeroExponent = 45.0;

__global__ __launch_bounds__(kFW, 2) void k_rbf_fit(const double* __restrict__ layers, const double* __restrict__ vel,
                                                 const double* __restrict__ w, const int32_t* __restrict__ off,
                                                 int M, int P, int nmax, double eps, double* __restrict__ coeffs,
                                                 double* __restrict__ tiles, size_t slot_doubles) {
  // LDS: A and B (32 x 32 tiles), then y (later c) of both components, one double2 per padded node
  extern __shared__ double pool[];
  double* A = pool;
  double* B = pool + kT * kLd;
  double2* yv = reinterpret_cast<double2*>(pool + 2 * kT * kLd);

  const int lane = threadIdx.x, i16 = lane & 15, k4 = lane >> 4;
  double2* slot = reinterpret_cast<double2*>(tiles + (size_t)blockIdx.x * slot_doubles);
  constexpr int kTile2 = kT * kT / 2;  // double2 per tile
  const size_t P5 = (size_t)5 * P;

  for (int v = blockIdx.x; v < M; v += gridDim.x) {
    const int j0 = clamp_i(off[v], 0, P);
    const int j1 = max(j0, clamp_i(off[v + 1], 0, P));
    const int npts = j1 - j0;
    if (npts == 0) continue;
    const int n = 5 * npts;
    double* cx = coeffs + (size_t)5 * j0;
    double* cy = coeffs + P5 + (size_t)5 * j0;
    if (npts > nmax) {
      for (int a = lane; a < n; a += kFW) {
        cx[a] = NAN;
        cy[a] = NAN;
      }
      continue;
    }
    const double h = wave_mean_spacing(w + j0, npts);
    NodeView nv;
    nv.x = layers + (size_t)5 * j0;
    nv.y = layers + P5 + (size_t)5 * j0;
    const double* ux = vel + (size_t)5 * j0;
    const double* uy = vel + P5 + (size_t)5 * j0;
    nv.n = n;
    nv.npts = npts;
    nv.inv_w2 = 1.0 / ((eps * h) * (eps * h));
    const int nb = (n + kT - 1) / kT;

    // first tile column of every tile row (lane I: tile row I), from the bounding boxes of the tiles' nodes; a
    // distance that is not a number counts as near
    int fcol = 0;
    {
      wave_sync();  // LDS is free
      double xl = INFINITY, xh = -INFINITY, yl = INFINITY, yh = -INFINITY;
      if (lane < nb)
        for (int b = lane * kT; b < min(n, (lane + 1) * kT); ++b) {
          const int a = node_index(b, npts);
          xl = fmin(xl, nv.x[a]);
          xh = fmax(xh, nv.x[a]);
          yl = fmin(yl, nv.y[a]);
          yh = fmax(yh, nv.y[a]);
        }
      if (lane < nb) {
        A[4 * lane] = xl;
        A[4 * lane + 1] = xh;
        A[4 * lane + 2] = yl;
        A[4 * lane + 3] = yh;
      }
      wave_sync();
      if (lane < nb)
        for (; fcol < lane; ++fcol) {
          const double dx = fmax(0.0, fmax(xl - A[4 * fcol + 1], A[4 * fcol] - xh));
          const double dy = fmax(0.0, fmax(yl - A[4 * fcol + 3], A[4 * fcol + 2] - yh));
          if (!((dx * dx + dy * dy) * nv.inv_w2 > kZeroExponent)) break;
        }
    }

    // ---- factorisation and forward substitution, panel by panel
#pragma unroll 1
    for (int J = 0; J < nb; ++J) {
      const int fJ = __builtin_amdgcn_readlane(fcol, J);
      double2 ps[2] = {make_double2(0.0, 0.0), make_double2(0.0, 0.0)};  // sum_k L_Jk y_k, rows 16 R + i16
      Tile W;
      {
        Acc acc;
        minus_entries<true>(acc, nv, J, J, lane);
#pragma unroll 1
        for (int k = fJ; k < J; ++k) {
          const Tile l = load_tile(slot + tile_index(J, k) * kTile2, lane);
          tile_gemm<true>(acc, l, l);
#pragma unroll
          for (int s = 0; s < 8; ++s) {
            const double2 yk = yv[k * kT + 4 * s + k4];
#pragma unroll
            for (int R = 0; R < 2; ++R) {
              ps[R].x = fma(l.e[R][s], yk.x, ps[R].x);
              ps[R].y = fma(l.e[R][s], yk.y, ps[R].y);
            }
          }
        }
        wave_sync();  // A and B are free
        minus_to_lds<true>(A, acc, lane);
        wave_sync();
        factor_invert(A, B, lane);
        W = tile_from_lds(B, lane);
        store_tile(slot + tile_index(J, J) * kTile2, lane, W);
      }
      {  // y_J = W (u_J - sum): the residual goes through A's first rows
        double2* tv = reinterpret_cast<double2*>(A);
#pragma unroll
        for (int R = 0; R < 2; ++R) {
          for (int o = 16; o < 64; o <<= 1) {
            ps[R].x += __shfl_xor(ps[R].x, o);
            ps[R].y += __shfl_xor(ps[R].y, o);
          }
          const int b = J * kT + 16 * R + i16;
          if (k4 == R) {
            const int a = node_index(min(b, n - 1), npts);
            tv[16 * R + i16] = b < n ? make_double2(ux[a] - ps[R].x, uy[a] - ps[R].y) : make_double2(0.0, 0.0);
          }
        }
        wave_sync();
        double2 yj[2] = {make_double2(0.0, 0.0), make_double2(0.0, 0.0)};
#pragma unroll
        for (int s = 0; s < 8; ++s) {
          const double2 t = tv[4 * s + k4];
#pragma unroll
          for (int R = 0; R < 2; ++R) {
            yj[R].x = fma(W.e[R][s], t.x, yj[R].x);
            yj[R].y = fma(W.e[R][s], t.y, yj[R].y);
          }
        }
#pragma unroll
        for (int R = 0; R < 2; ++R) {
          for (int o = 16; o < 64; o <<= 1) {
            yj[R].x += __shfl_xor(yj[R].x, o);
            yj[R].y += __shfl_xor(yj[R].y, o);
          }
          if (k4 == R) yv[J * kT + 16 * R + i16] = yj[R];
        }
        wave_sync();
      }
#pragma unroll 1
      for (int I = J + 1; I < nb; ++I) {
        const int fI = __builtin_amdgcn_readlane(fcol, I);
        if (fI > J) continue;
        Acc acc;
        minus_entries<false>(acc, nv, I, J, lane);
#pragma unroll 1
        for (int k = max(fI, fJ); k < J; ++k) {  // T = K - sum_k L_Ik L_Jk^T
          const Tile a = load_tile(slot + tile_index(I, k) * kTile2, lane);
          const Tile b = load_tile(slot + tile_index(J, k) * kTile2, lane);
          tile_gemm<false>(acc, a, b);
        }
        wave_sync();  // A is free
        minus_to_lds<false>(A, acc, lane);
        wave_sync();
        const Tile t = tile_from_lds(A, lane);
        Acc out;  // L_IJ = T W^T; W's upper right block is zero
#pragma unroll
        for (int R = 0; R < 2; ++R)
#pragma unroll
          for (int C = 0; C < 2; ++C) out[R][C] = double4v{0.0, 0.0, 0.0, 0.0};
#pragma unroll
        for (int s = 0; s < 8; ++s)
#pragma unroll
          for (int R = 0; R < 2; ++R) {
            if (s < 4) out[R][0] = __builtin_amdgcn_mfma_f64_16x16x4f64(t.e[R][s], W.e[0][s], out[R][0], 0, 0, 0);
            out[R][1] = __builtin_amdgcn_mfma_f64_16x16x4f64(t.e[R][s], W.e[1][s], out[R][1], 0, 0, 0);
          }
        wave_sync();  // the reads of A are done
#pragma unroll
        for (int R = 0; R < 2; ++R)
#pragma unroll
          for (int C = 0; C < 2; ++C)
#pragma unroll
            for (int q = 0; q < 4; ++q) A[acc_row(lane, R, q) * kLd + acc_col(lane, C)] = out[R][C][q];
        wave_sync();
        store_tile(slot + tile_index(I, J) * kTile2, lane, tile_from_lds(A, lane));
      }
    }

    // ---- back substitution: c_J = W_JJ^T (y_J - sum_{I > J} L_IJ^T c_I).  Lane (i16, k4) adds rows i16 and 16 + i16
    // of columns 4 s + k4; the 16 lanes of a row are added at the end of each sum.
    auto add_rows = [](const Tile& t, const double2* __restrict__ c, int i16, double2 (&z)[8]) {
      const double2 c0 = c[i16], c1 = c[16 + i16];
#pragma unroll
      for (int s = 0; s < 8; ++s) {
        z[s].x = fma(t.e[1][s], c1.x, fma(t.e[0][s], c0.x, z[s].x));
        z[s].y = fma(t.e[1][s], c1.y, fma(t.e[0][s], c0.y, z[s].y));
      }
    };
#pragma unroll 1
    for (int J = nb - 1; J >= 0; --J) {
      double2 z[8];
#pragma unroll
      for (int s = 0; s < 8; ++s) z[s] = make_double2(0.0, 0.0);
      const Tile W = load_tile(slot + tile_index(J, J) * kTile2, lane);
#pragma unroll 1
      for (int I = J + 1; I < nb; ++I) {
        if (__builtin_amdgcn_readlane(fcol, I) > J) continue;
        add_rows(load_tile(slot + tile_index(I, J) * kTile2, lane), yv + I * kT, i16, z);
      }
      double2* tv = reinterpret_cast<double2*>(A);
      wave_sync();  // A is free
#pragma unroll
      for (int s = 0; s < 8; ++s) {
        z[s].x = row_sum(z[s].x);
        z[s].y = row_sum(z[s].y);
        if (i16 == s) {
          const double2 y = yv[J * kT + 4 * s + k4];
          tv[4 * s + k4] = make_double2(y.x - z[s].x, y.y - z[s].y);
        }
        z[s] = make_double2(0.0, 0.0);
      }
      wave_sync();
      add_rows(W, tv, i16, z);
#pragma unroll
      for (int s = 0; s < 8; ++s) {
        z[s].x = row_sum(z[s].x);
        z[s].y = row_sum(z[s].y);
        if (i16 == s) yv[J * kT + 4 * s + k4] = z[s];
      }
      wave_sync();
    }
    // a pivot or value that was not a number makes all of its component's coefficients so (a skipped tile may have
    // kept it from some of them)
    bool badx = false, bady = false;
    for (int b = lane; b < n; b += kFW) {
      const double2 c = yv[b];
      badx |= c.x != c.x;
      bady |= c.y != c.y;
    }
    badx = __any(badx);
    bady = __any(bady);
    for (int b = lane; b < n; b += kFW) {
      const double2 c = yv[b];
      const int a = node_index(b, npts);
      cx[a] = badx ? NAN : c.x;
      cy[a] = bady ? NAN : c.y;
    }
    wave_sync();
  }
}

constexpr int kEB = 256;  // threads of the evaluation kernel: 4 wavefronts, one pair each

__global__ __launch_bounds__(kEB) void k_rbf_eval_near(const double* __restrict__ layers,
                                                       const double* __restrict__ coeffs,
                                                       const double* __restrict__ w, const int32_t* __restrict__ off,
                                                       int M, int P, double eps, const double* __restrict__ tg,
                                                       int n_targets, const int32_t* __restrict__ pairs,
                                                       const int32_t* __restrict__ count, int capacity,
                                                       double* __restrict__ out) {
  const int lane = threadIdx.x & 63;
  const int waves = gridDim.x * (kEB / 64);
  const int npairs = min(max(*count, 0), capacity);
  const size_t P5 = (size_t)5 * P;
  for (int k = blockIdx.x * (kEB / 64) + (threadIdx.x >> 6); k < npairs; k += waves) {
    const int i = pairs[2 * k];
    const int v = pairs[2 * k + 1];
    if (i < 0 || i >= n_targets || v < 0 || v >= M) continue;  // not a pair of this problem
    const int j0 = clamp_i(off[v], 0, P);
    const int j1 = max(j0, clamp_i(off[v + 1], 0, P));
    const int npts = j1 - j0;
    if (npts == 0) continue;
    const double h = wave_mean_spacing(w + j0, npts);
    const double inv_w2 = 1.0 / ((eps * h) * (eps * h));
    const double px = tg[i], py = tg[n_targets + i];
    const double* nx = layers + (size_t)5 * j0;
    const double* ny = layers + P5 + (size_t)5 * j0;
    const double* cx = coeffs + (size_t)5 * j0;
    const double* cy = coeffs + P5 + (size_t)5 * j0;
    double sx = 0.0, sy = 0.0;
    for (int a = lane; a < 5 * npts; a += 64) {
      const double dx = px - nx[a];
      const double dy = py - ny[a];
      const double g = exp(-(dx * dx + dy * dy) * inv_w2);
      sx = fma(g, cx[a], sx);
      sy = fma(g, cy[a], sy);
    }
#pragma unroll
    for (int m = 32; m >= 1; m >>= 1) {
      sx += __shfl_xor(sx, m, 64);
      sy += __shfl_xor(sy, m, 64);
    }
    if (lane == 0) {
      atomicAdd(out + i, sx);
      atomicAdd(out + n_targets + i, sy);
    }
  }
}

}  // namespace

// Doubles of a vesicle's slot.  The lower tiles take nb (nb + 1) / 2 of them; nb tiles and two vectors more are the size
// that callers of the C interface have met, and it stays what a workspace is measured by.
size_t rbf_slot_doubles(int nmax) {
  const int nb = (5 * nmax + kT - 1) / kT;
  return (size_t)nb * (nb + 3) / 2 * (kT * kT) + (size_t)2 * nb * kT;
}

hipError_t launch_rbf_fit(const double* layers, const double* vel, const double* w, const int32_t* off, int M, int P,
                          int nmax, double eps, double* coeffs, double* tiles, int slots, void* stream) {
  if (M == 0 || P == 0) return hipSuccess;
  if (5 * nmax > kMaxNodes || slots < 1) return hipErrorInvalidValue;
  const int grid = M < slots ? M : slots;
  const size_t lds = sizeof(double) * (size_t)(2 * kT * kLd + 2 * kT * ((5 * nmax + kT - 1) / kT));
  hipLaunchKernelGGL(k_rbf_fit, dim3(grid), dim3(kFW), lds, reinterpret_cast<hipStream_t>(stream), layers, vel, w, off,
                     M, P, nmax, eps, coeffs, tiles, rbf_slot_doubles(nmax));
  return hipGetLastError();
}

hipError_t launch_rbf_eval_near(const double* layers, const double* coeffs, const double* w, const int32_t* off,
                                int M, int P, double eps, const double* targets, int n_targets, const int32_t* pairs,
                                const int32_t* count, int capacity, double* out, void* stream) {
  if (capacity == 0 || M == 0 || P == 0 || n_targets == 0) return hipSuccess;
  const int need = (capacity + kEB / 64 - 1) / (kEB / 64);
  const int grid = need < 4096 ? need : 4096;
  hipLaunchKernelGGL(k_rbf_eval_near, dim3(grid), dim3(kEB), 0, reinterpret_cast<hipStream_t>(stream), layers, coeffs,
                     w, off, M, P, eps, targets, n_targets, pairs, count, capacity, out);
  return hipGetLastError();
}

}  // namespace vesnet

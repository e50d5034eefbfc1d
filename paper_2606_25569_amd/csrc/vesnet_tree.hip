// Tree far fields on gfx950: the far-field sum of eq. (single_layer) at O(P log P) (treecode) and O(P)
// (fast multipole method) cost.  The paper evaluates the sum directly, names the fast multipole method as
// the route to O(M) cost and leaves fast summation out of scope (Section 4.1); both methods here are fast,
// approximate alternatives with their own accuracy contract (order p of the expansions).
//
// With complex numbers z = x + i y, F_j = w_j (f_x + i f_y)_j, u = u_x + i u_y, each Stokeslet term is
//   -F_j ln|z - z_j| + F_j / 2 + (z - z_j) conj(F_j / (z - z_j)) / 2,
// so a box of sources with centre c, zeta_j = z_j - c, acts at w = z - c, t = 1/w, through the
// power moments M_k[q] = sum_j q_j zeta_j^k of three charge sets (F, conj F, conj(zeta) F):
//   -M_0[F] ln|w| + 1/2 sum_{k=1}^p (M_k[F] t^k + conj(M_k[conj F] t^k)) / k + M_0[F] / 2
//   + (w conj(Phi) - conj(Psi)) / 2,   Phi = sum_{k=0}^p M_k[F] t^(k+1),  Psi = sum_k M_k[conj(zeta) F] t^(k+1).
//
// Tree: a uniform quadtree of depth L over the bounding square of the points.  Leaf moments come from
// the points (k_tc_p2m), coarser ones by exact binomial translation (k_tc_m2m).  A target takes, at each
// level l = 2..L, the interaction list of its level-l ancestor (children of the parent's 3 x 3
// neighbourhood not adjacent to the ancestor) through the expansions, and the 3 x 3 leaves around its own
// directly, skipping its own vesicle; own-vesicle sources outside those leaves, which the expansions
// included, are subtracted exactly (own_terms).  Everything is FP64.
//
// Treecode: every target evaluates the series of every box of its lists (k_tc_eval); the
// evaluation merges the conj-F log series and Psi into one series D, and writes w conj(Phi) as
// (w / conj w) conj(E), E = sum_k M_k[F] t^k: three Horner chains per box.
// Fast multipole method: each box's series becomes a Taylor polynomial of degree p about the centre of
// every box whose list holds it (k_fmm_m2l, on the matrix cores), the polynomials of a leaf's ancestors
// are re-centred onto the leaf (k_fmm_l2l), and every target evaluates its leaf's polynomial
// (k_fmm_eval).
#include <hip/hip_runtime.h>
#include <math.h>
#include <stdint.h>

#include "vesnet_internal.h"

namespace vesnet {

namespace {

constexpr int kTB = 256;       // threads of the point-parallel kernels
constexpr int kBBoxBlocks = 256;
constexpr int kSortMax = 2048;  // larger leaves keep the order of the atomic scatter

struct Geom {
  double x0, y0, side;  // lower-left corner and side of the root square
};

constexpr int kMaxDepth = 10;
constexpr int kMaxOrder = 48;

// Where each level's boxes start: in boxes (counts) and in complex moment entries.
struct Levels {
  unsigned long long box[kMaxDepth + 1];
  unsigned long long mom[kMaxDepth + 1];
};

__device__ __forceinline__ int clamp_i(int x, int lo, int hi) { return x < lo ? lo : (x > hi ? hi : x); }

__device__ __forceinline__ double2 cmul(double2 a, double2 b) {
  return make_double2(fma(a.x, b.x, -a.y * b.y), fma(a.x, b.y, a.y * b.x));
}
// a * t + c
__device__ __forceinline__ double2 cfma(double2 a, double2 t, double2 c) {
  return make_double2(fma(a.x, t.x, fma(-a.y, t.y, c.x)), fma(a.x, t.y, fma(a.y, t.x, c.y)));
}

// Box centre at a level with n boxes per side (contraction off: the same bits as the plain formula).
__device__ __forceinline__ double2 box_center(const Geom& g, int n, int bx, int by) {
#pragma clang fp contract(off)
  const double wl = g.side / (double)n;
  return make_double2(g.x0 + ((double)bx + 0.5) * wl, g.y0 + ((double)by + 0.5) * wl);
}

// First box of level l >= 2 when levels 2, 3, ... are stored one after another: sum_{m=2}^{l-1} 4^m.
__device__ __forceinline__ size_t level_box_base(int l) { return (((size_t)1 << (2 * l)) - 16) / 3; }

// ---------------------------------------------------------------- tree construction

// Binomial table: entry [m - 1][l] = C(m + l - 1, l), m = 1 .. kTabM, l = 0 .. kTabL - 1, over the whole padded range
// that the matrix-core tiles read, by Pascal's rule (sums of integers, exact below 2^53), made by the compiler.
constexpr int kTabL = 64;
constexpr int kTabM = 4 * ((kMaxOrder + 1 + 3) / 4);  // m up to 4 ceil((p + 1) / 4)
struct Binomials {
  double t[kTabM][kTabL];
  constexpr Binomials() : t() {
    for (int m = 0; m < kTabM; ++m)
      for (int l = 0; l < kTabL; ++l) t[m][l] = m == 0 || l == 0 ? 1.0 : t[m - 1][l] + t[m][l - 1];
  }
};
__device__ constexpr Binomials kBinomials{};

// Bounding boxes of the points' parts.  Also builds the evaluation's log table when tab is not null, clears the leaf
// counters, and with count given the near-field list's count and status.
__global__ __launch_bounds__(kTB) void k_tc_bbox_partial(const double* __restrict__ X, int P,
                                                         double* __restrict__ part, double2* __restrict__ tab,
                                                         int32_t* __restrict__ counts,
                                                         int nleaf, int32_t* __restrict__ count,
                                                         int32_t* __restrict__ flag) {
  __shared__ double red[4][kTB];
  for (int e = blockIdx.x * kTB + threadIdx.x; e < nleaf; e += gridDim.x * kTB) counts[e] = 0;
  if (count != nullptr && blockIdx.x == 0 && threadIdx.x == 0) *count = *flag = 0;
  if (tab != nullptr)
    for (int e = blockIdx.x * kTB + threadIdx.x; e < kHalfLogTab; e += gridDim.x * kTB) tab[e] = half_log_entry(e);
  double xl = INFINITY, xh = -INFINITY, yl = INFINITY, yh = -INFINITY;
  for (int j = blockIdx.x * kTB + threadIdx.x; j < P; j += gridDim.x * kTB) {
    const double x = X[j], y = X[P + j];
    xl = fmin(xl, x);
    xh = fmax(xh, x);
    yl = fmin(yl, y);
    yh = fmax(yh, y);
  }
  red[0][threadIdx.x] = xl;
  red[1][threadIdx.x] = xh;
  red[2][threadIdx.x] = yl;
  red[3][threadIdx.x] = yh;
  __syncthreads();
  for (int s = kTB / 2; s > 0; s >>= 1) {
    if (threadIdx.x < s) {
      red[0][threadIdx.x] = fmin(red[0][threadIdx.x], red[0][threadIdx.x + s]);
      red[1][threadIdx.x] = fmax(red[1][threadIdx.x], red[1][threadIdx.x + s]);
      red[2][threadIdx.x] = fmin(red[2][threadIdx.x], red[2][threadIdx.x + s]);
      red[3][threadIdx.x] = fmax(red[3][threadIdx.x], red[3][threadIdx.x + s]);
    }
    __syncthreads();
  }
  if (threadIdx.x < 4) part[blockIdx.x * 4 + threadIdx.x] = red[threadIdx.x][0];
}

// The root square of the parts' bounding boxes, by one wavefront; the value is lane 0's.
__device__ __forceinline__ Geom root_square(const double* __restrict__ part, int nparts) {
  const int lane = threadIdx.x & 63;
  double xl = INFINITY, xh = -INFINITY, yl = INFINITY, yh = -INFINITY;
  for (int b = lane; b < nparts; b += 64) {
    xl = fmin(xl, part[4 * b]);
    xh = fmax(xh, part[4 * b + 1]);
    yl = fmin(yl, part[4 * b + 2]);
    yh = fmax(yh, part[4 * b + 3]);
  }
#pragma unroll
  for (int m = 32; m >= 1; m >>= 1) {
    xl = fmin(xl, __shfl_xor(xl, m, 64));
    xh = fmax(xh, __shfl_xor(xh, m, 64));
    yl = fmin(yl, __shfl_xor(yl, m, 64));
    yh = fmax(yh, __shfl_xor(yh, m, 64));
  }
  Geom g;
  {
#pragma clang fp contract(off)
    double side = fmax(xh - xl, yh - yl);
    if (side == 0.0) side = 1.0;
    g.x0 = 0.5 * (xl + xh) - 0.5 * side;
    g.y0 = 0.5 * (yl + yh) - 0.5 * side;
    g.side = side;
  }
  return g;
}

__global__ __launch_bounds__(64) void k_tc_zero(int32_t* __restrict__ a) {
  if (threadIdx.x == 0) *a = 0;
}

// Within a wavefront, the lanes of equal keys form a group: one atomic adds the group's size to counter[key] and returns
// the group's base, and each lane takes base + its rank among the group's lanes.  Consecutive points mostly share a
// leaf, so a wavefront needs a few atomics instead of 64; they are issued together.
__device__ __forceinline__ int wave_group_add(bool ok, int key, int32_t* __restrict__ counter) {
  const int lane = threadIdx.x & 63;
  unsigned long long todo = __ballot(ok), group = 0;
  while (todo) {
    const int lk = __shfl(key, __ffsll(todo) - 1);
    const unsigned long long same = __ballot(ok && key == lk);  // not yet placed: earlier groups had other keys
    if ((same >> lane) & 1ull) group = same;
    todo &= ~same;
  }
  const int leader = __ffsll(group) - 1;
  int base = 0;
  if (ok && lane == leader) base = atomicAdd(counter + key, __popcll(group));
  base = __shfl(base, max(leader, 0));
  return base + __popcll(group & ((1ull << lane) - 1ull));
}

// Leaf of every point, its place in the leaf and the leaf occupancies in the first `pblocks` workgroups, which also
// clear the output; vesicle id of every point in the others, one workgroup per vesicle, which writes its index over its
// range (offsets clamped).
// With h2 given, also the squared near-field radius h_v^2 of every vesicle, h_v = sum_j w_j / N_v (the
// mean arclength spacing, summed in a fixed order), and bit 1 of *flag when h_v exceeds the leaf width
// (then a point within h_v of a target may lie outside its 3 x 3 leaves).
// Every workgroup that needs the root square forms it from the parts' boxes itself: a launch of its own for it, one for
// the ids and one to clear the counters cost 4 us each.
__global__ __launch_bounds__(kTB) void k_tc_leaf(const double* __restrict__ X, int P, const double* __restrict__ part,
                                                 int nparts, int pblocks, int depth, Geom* __restrict__ geom,
                                                 int32_t* __restrict__ leafid, int32_t* __restrict__ counts,
                                                 int32_t* __restrict__ place,
                                                 const int32_t* __restrict__ off, int32_t* __restrict__ vid,
                                                 const double* __restrict__ w, double* __restrict__ h2,
                                                 int32_t* __restrict__ flag, double* __restrict__ out) {
  __shared__ Geom root;
  __shared__ double red[kTB];
  const bool points = (int)blockIdx.x < pblocks;
  if (points || h2 != nullptr) {
    if (threadIdx.x < 64) {
      const Geom g = root_square(part, nparts);
      if (threadIdx.x == 0) {
        root = g;
        if (blockIdx.x == 0) *geom = g;
      }
    }
    __syncthreads();
  }
  const int n = 1 << depth;
  if (points) {
    const Geom g = root;
    for (int j0 = blockIdx.x * kTB; j0 < P; j0 += pblocks * kTB) {  // the same trip count for every lane
      const int j = j0 + (int)threadIdx.x;
      const bool ok = j < P;
      int leaf = 0;
      if (ok) {
        int ix, iy;
        {
#pragma clang fp contract(off)
          const double wl = g.side / (double)n;
          ix = clamp_i((int)floor((X[j] - g.x0) / wl), 0, n - 1);
          iy = clamp_i((int)floor((X[P + j] - g.y0) / wl), 0, n - 1);
        }
        leaf = ix * n + iy;
        leafid[j] = leaf;
        out[j] = out[P + j] = 0.0;
      }
      const int at = wave_group_add(ok, leaf, counts);
      if (ok) place[j] = at;
    }
    return;
  }
  const int v = blockIdx.x - pblocks;
  const int v0 = clamp_i(off[v], 0, P), v1 = max(v0, clamp_i(off[v + 1], 0, P));
  for (int j = v0 + (int)threadIdx.x; j < v1; j += kTB) vid[j] = v;
  if (h2 == nullptr) return;
  double a = 0.0;
  for (int j = v0 + (int)threadIdx.x; j < v1; j += kTB) a += w[j];
  red[threadIdx.x] = a;
  __syncthreads();
  for (int s = kTB / 2; s > 0; s >>= 1) {
    if ((int)threadIdx.x < s) red[threadIdx.x] += red[threadIdx.x + s];
    __syncthreads();
  }
  if (threadIdx.x == 0) {
    const double h = v1 > v0 ? red[0] / (double)(v1 - v0) : 0.0;
    h2[v] = h * h;
    if (h > root.side / (double)n) atomicOr(flag, 2);
  }
}

// Exclusive scans of the leaf occupancies (starts) and of their chunks of 2^cshift targets (wave starts), by one
// workgroup: 4,096 leaves at a time, four consecutive ones a thread, each wavefront's sums by shuffles and the sixteen
// wavefronts' through LDS.  Latency bounds it: depth 6 6.8 -> 4.8 us, depth 7 34 -> 7.2 (before: every thread walked its
// leaves one by one, ten rounds of two barriers).
__global__ __launch_bounds__(1024) void k_tc_scan(const int32_t* __restrict__ counts, int nleaf,
                                                  int32_t* __restrict__ starts, int32_t* __restrict__ wstart,
                                                  int cshift) {
  __shared__ int2 total[2][16];  // of the wavefronts, alternating between passes
  const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
  const int up = (1 << cshift) - 1;
  const auto load = [&](int i) {
    if (i + 4 <= nleaf) return *reinterpret_cast<const int4*>(counts + i);
    return make_int4(i < nleaf ? counts[i] : 0, i + 1 < nleaf ? counts[i + 1] : 0, i + 2 < nleaf ? counts[i + 2] : 0, 0);
  };
  const auto store = [&](int32_t* __restrict__ to, int i, int first, int x, int y, int z) {
    const int4 v = make_int4(first, first + x, first + x + y, first + x + y + z);
    if (i + 4 <= nleaf) {
      *reinterpret_cast<int4*>(to + i) = v;
    } else {
      if (i < nleaf) to[i] = v.x;
      if (i + 1 < nleaf) to[i + 1] = v.y;
      if (i + 2 < nleaf) to[i + 2] = v.z;
    }
  };
  int a0 = 0, b0 = 0;  // sums of the earlier passes
  int4 next = load(4 * t);
  for (int base = 0, pass = 0; base < nleaf; base += 4096, pass ^= 1) {
    const int4 c = next;
    next = load(base + 4096 + 4 * t);
    const int4 d = make_int4((c.x + up) >> cshift, (c.y + up) >> cshift, (c.z + up) >> cshift, (c.w + up) >> cshift);
    const int own_a = c.x + c.y + c.z + c.w, own_b = d.x + d.y + d.z + d.w;
    int a = own_a, b = own_b;
    for (int o = 1; o < 64; o <<= 1) {  // inclusive over the wavefront
      const int xa = __shfl_up(a, o), xb = __shfl_up(b, o);
      if (lane >= o) {
        a += xa;
        b += xb;
      }
    }
    if (lane == 63) total[pass][wave] = make_int2(a, b);
    __syncthreads();
    int ea = a0 + a - own_a, eb = b0 + b - own_b;
#pragma unroll
    for (int q = 0; q < 16; ++q) {
      const int2 w = total[pass][q];
      if (q < wave) {
        ea += w.x;
        eb += w.y;
      }
      a0 += w.x;
      b0 += w.y;
    }
    store(starts, base + 4 * t, ea, c.x, c.y, c.z);
    store(wstart, base + 4 * t, eb, d.x, d.y, d.z);
  }
  if (t == 0) {
    starts[nleaf] = a0;
    wstart[nleaf] = b0;
  }
}

// Every point to its place in its leaf (the order of the atomics).
__global__ __launch_bounds__(kTB) void k_tc_scatter(const int32_t* __restrict__ leafid, int P,
                                                    const int32_t* __restrict__ starts,
                                                    const int32_t* __restrict__ place, int32_t* __restrict__ perm) {
  for (int j = blockIdx.x * kTB + threadIdx.x; j < P; j += gridDim.x * kTB) perm[starts[leafid[j]] + place[j]] = j;
}

// Points of each leaf in ascending index order (deterministic sums).  One wavefront per leaf: the
// keys (distinct point indices) go to LDS and each is written at its rank, the number of smaller
// keys in the leaf.  The points' records (x, y, w f_x, w f_y) and vesicle ids are stored in the same order: later
// kernels read whole leaves contiguously instead of gathering five arrays through the permutation.
__global__ __launch_bounds__(64) void k_tc_sort(const double* __restrict__ X, const double* __restrict__ f,
                                                const double* __restrict__ w, int P, const int32_t* __restrict__ vid,
                                                const int32_t* __restrict__ starts, int32_t* __restrict__ perm,
                                                double4* __restrict__ srec, int32_t* __restrict__ svid) {
  __shared__ int32_t key[kSortMax];
  const int leaf = blockIdx.x;
  const int s0 = starts[leaf], n = starts[leaf + 1] - s0;
  const bool sort = n <= kSortMax;
  if (sort) {
    for (int a = threadIdx.x; a < n; a += 64) key[a] = perm[s0 + a];
    __syncthreads();
  }
  for (int a = threadIdx.x; a < n; a += 64) {
    const int32_t j = sort ? key[a] : perm[s0 + a];
    const double4 rec = make_double4(X[j], X[P + j], w[j] * f[j], w[j] * f[P + j]);  // on its way during the ranking
    const int32_t id = vid[j];
    int slot = s0 + a;
    if (sort) {
      int rank = 0;
      for (int b = 0; b < n; ++b) rank += key[b] < j;
      slot = s0 + rank;
      perm[slot] = j;
    }
    srec[slot] = rec;
    svid[slot] = id;
  }
}

// ---------------------------------------------------------------- moments
//
// Moments of a box: 4 rows of (p + 1) complex numbers: row 0 M_k[F], row 1 M_k[conj F] (divided by k
// for k >= 1 once all translations are done), row 2 M_k[conj(zeta) F], row 3 M_k[F] / k (filled last).

typedef double double4v __attribute__((ext_vector_type(4)));

// The value of the neighbouring lane (lanes 2 i and 2 i + 1 exchange).
__device__ __forceinline__ double quad_swap(double v) {
  const int lo = __builtin_amdgcn_update_dpp(0, __double2loint(v), 0xB1, 0xF, 0xF, false);  // quad_perm 1, 0, 3, 2
  const int hi = __builtin_amdgcn_update_dpp(0, __double2hiint(v), 0xB1, 0xF, 0xF, false);
  return __hiloint2double(hi, lo);
}

// The value two lanes up, and of the other half, in each row of 16 lanes.
template <int kCtrl>
__device__ __forceinline__ double row_move(double v) {
  const int lo = __builtin_amdgcn_update_dpp(0, __double2loint(v), kCtrl, 0xF, 0xF, true);
  const int hi = __builtin_amdgcn_update_dpp(0, __double2hiint(v), kCtrl, 0xF, 0xF, true);
  return __hiloint2double(hi, lo);
}
__device__ __forceinline__ double row_shift2(double v) { return row_move<0x102>(v); }  // row_shl:2
__device__ __forceinline__ double row_half(double v) { return row_move<0x128>(v); }    // row_ror:8

// x^k for 0 <= k < 64.
__device__ __forceinline__ double pow_int(double x, int k) {
  double r = 1.0;
#pragma unroll
  for (int b = 0; b < 6; ++b) {
    if (k & (1 << b)) r *= x;
    x *= x;
  }
  return r;
}

__device__ __forceinline__ double2 cpow_int(double2 x, int k) {
  double2 r = make_double2(1.0, 0.0);
#pragma unroll
  for (int b = 0; b < 6; ++b) {
    const double2 t = cmul(r, x);
    if (k & (1 << b)) r = t;
    x = cmul(x, x);
  }
  return r;
}

// e^(i pi a / 4).
__device__ __forceinline__ double2 eighth_turn(int a) {
  constexpr double h = 0.70710678118654752440;
  const auto cosine = [&](int t) {
    const int m = t & 3;
    const double c = m == 0 ? 1.0 : (m == 1 ? h : (m == 2 ? 0.0 : -h));
    return (t & 4) ? -c : c;
  };
  return make_double2(cosine(a), cosine(a + 6));
}

// A box's moments re-centred to its parent's centre, d = box centre - parent centre:
//   M'_k = sum_{m <= k} C(k, m) d^(k-m) M_m = d^k sum_m C(k, m) (d^-m M_m)
// (and the conj(zeta) F row gains conj(d) times the translated F row: left to the sum over the children), by one
// wavefront on the matrix cores: the triangle of binomials, which every box shares, stays in registers as the first
// operand, and the six real columns of d^-m M_m (three rows, Re and Im) are the second.  For 8 K >= p + 1 orders.
// d = delta e^(i pi a / 4), a = 1, 3, 5, 7, so its powers are real powers and eighths of a turn.  The division by
// delta^m takes the power of two of delta apart, which scales exactly, and the rest lies in [1/2, 1): the quotients
// overflow only where the moments in units of the box do, and the orders above p, which hold zeros, cannot turn into
// zero times infinity.
// (On the vector units, a lane per order, the moments' broadcasts from LDS bounded it: 5.5 us for 64 boxes on a CU.)
template <int K>
struct Recentre {
  static constexpr int kTiles = (K + 1) / 2, kOrders = 8 * K, kLds = 8 * kOrders;  // LDS doubles of run()
  static constexpr int steps(int rt) { return 4 * (rt + 1) < 2 * K ? 4 * (rt + 1) : 2 * K; }
  double a[kTiles][2 * K];
  int lane, p;

  __device__ __forceinline__ explicit Recentre(int order) : lane(threadIdx.x & 63), p(order) {
#pragma unroll
    for (int rt = 0; rt < kTiles; ++rt)
#pragma unroll
      for (int s = 0; s < steps(rt); ++s) {
        const int k = 16 * rt + (lane & 15), m = min(4 * s + (lane >> 4), kTabM - 1);
        const double c = kBinomials.t[m][max(k - m, 0)];
        a[rt][s] = m <= k ? c : 0.0;
      }
  }

  // d^k, d = delta e^(i pi turn / 4).
  __device__ __forceinline__ static double2 power(double delta, int turn, int k) {
    const double2 e = eighth_turn(turn * k);
    const double r = pow_int(delta, k);
    return make_double2(r * e.x, r * e.y);
  }

  // m0, m1, m2: lane m's moments of order m (0 beyond p).  pw (LDS): d^0 .. d^p.  x (LDS): kLds doubles of this
  // wavefront, where it leaves the translated rows, [3][p + 1] complex.
  __device__ __forceinline__ void run(double2 m0, double2 m1, double2 m2, double delta, int turn,
                                      const double2* __restrict__ pw, double* __restrict__ x) const {
    if (lane < kOrders) {
      int ex;
      const double r = pow_int(1.0 / frexp(delta, &ex), lane);
      const double2 e = eighth_turn(-turn * lane);
      const auto put = [&](int c, double2 m) {
        const double2 t = cmul(m, e);
        x[8 * lane + 2 * c] = ldexp(t.x, -ex * lane) * r;
        x[8 * lane + 2 * c + 1] = ldexp(t.y, -ex * lane) * r;
      };
      put(0, m0);
      put(1, m1);
      put(2, m2);
    }
    wave_sync();
    double4v acc[kTiles];
#pragma unroll
    for (int rt = 0; rt < kTiles; ++rt) acc[rt] = double4v{0.0, 0.0, 0.0, 0.0};
#pragma unroll
    for (int s = 0; s < 2 * K; ++s) {
      const double b = x[8 * (4 * s + (lane >> 4)) + (lane & 7)];
#pragma unroll
      for (int rt = 0; rt < kTiles; ++rt)
        if (s < steps(rt)) acc[rt] = __builtin_amdgcn_mfma_f64_16x16x4f64(a[rt][s], b, acc[rt], 0, 0, 0);
    }
    wave_sync();  // x is read
    const int c = lane & 15;
#pragma unroll
    for (int rt = 0; rt < kTiles; ++rt)
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const int k = 16 * rt + (lane >> 4) + 4 * v;
        const double2 e = pw[min(k, p)];
        const double mine = acc[rt][v], other = quad_swap(mine);  // Re and Im are neighbours
        if (c < 6 && k <= p) x[2 * ((c >> 1) * (p + 1) + k) + (c & 1)] = fma(mine, e.x, (c & 1) ? other * e.y : -(other * e.y));
      }
  }
};

// A parent's moments of order e mod (p + 1), row e / (p + 1), from the translated rows of its four children (kLds
// doubles apart): their sum in order, and for the conj(zeta) F row conj(d_q) times the F row of each.
__device__ __forceinline__ double2 children_sum(const double* __restrict__ x, int apart, int p, double half, int e) {
  double2 r = make_double2(0.0, 0.0);
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const double2* rows = reinterpret_cast<const double2*>(x + q * apart);
    double2 t = rows[e];
    if (e >= 2 * (p + 1)) t = cfma(make_double2(q & 2 ? half : -half, q & 1 ? -half : half), rows[e - 2 * (p + 1)], t);
    r.x += t.x;
    r.y += t.y;
  }
  return r;
}

// Child q's direction from its parent's centre in eighths of a turn (q & 2: right, q & 1: up).
__device__ __forceinline__ int child_turn(int q) { return (q & 2) ? ((q & 1) ? 1 : 7) : ((q & 1) ? 3 : 5); }

// Sums of pairs of lanes 32, 16 or 8 apart, of two values at once: the lanes with bit kOff clear get lo's, the others
// hi's.
template <int kOff>
__device__ __forceinline__ double pair_sums(double lo, double hi, int lane) {
  if constexpr (kOff == 8) {
    const bool up = lane & 8;
    const double keep = up ? hi : lo, send = up ? lo : hi;
    return keep + row_half(send);
  } else {
    const auto swap = [](unsigned x, unsigned y) {
      if constexpr (kOff == 32) return __builtin_amdgcn_permlane32_swap(x, y, false, false);
      else return __builtin_amdgcn_permlane16_swap(x, y, false, false);
    };
    const auto l = swap(__double2loint(lo), __double2loint(hi)), h = swap(__double2hiint(lo), __double2hiint(hi));
    return __hiloint2double(h[0], l[0]) + __hiloint2double(h[1], l[1]);
  }
}

__device__ __forceinline__ void direct_term(double zx, double zy, double sx, double sy, double Fx, double Fy,
                                            const double2* __restrict__ ltab, double& ux, double& uy) {
  const double rx = zx - sx, ry = zy - sy;
  const double q = rx * rx + ry * ry;
  const double lg = -0.5 * log_reduced(q, ltab);
  const double s = (rx * Fx + ry * Fy) * recip(q);
  ux = fma(lg, Fx, fma(s, rx, ux));
  uy = fma(lg, Fy, fma(s, ry, uy));
}

// Own-vesicle sources outside the 3 x 3 leaves around a target are in the expansions: their direct terms, to be
// subtracted.  A wavefront takes 64 consecutive targets of a vesicle and the vesicle's points 64 at a time.
// Neighbouring points share a leaf, so a chunk is a few runs of one leaf each: the first pass finds the runs, and each
// lane tests the runs and lists its far stretches of points (6% of the pairs at 2000 x 128, none for most vesicles of
// a shallow tree: then the chunk's records are not read at all).  The lanes' stretches are then evaluated side by side,
// as many steps as the longest list (38 us at 2000 x 128 with every lane testing every point, 21 by runs).  out of the
// wavefront's targets is written, -scale times their sum, where any of them has such terms.
constexpr int kOwnChunk = 64;
struct OwnLds {
  double2 ltab[kLogTab];
  double sx[kOwnChunk], sy[kOwnChunk], sfx[kOwnChunk], sfy[kOwnChunk];
  int32_t run0[kOwnChunk + 1], runl[kOwnChunk];  // first point and leaf of every run
  uint16_t lst[kOwnChunk / 2 + 1][64];           // lst[k][lane]: its k-th far stretch, begin | end << 8
};

__device__ void own_terms(OwnLds& m, const double* __restrict__ X, const double* __restrict__ f,
                          const double* __restrict__ w, int P, int v0, int v1, int t0,
                          const int32_t* __restrict__ leafid, int depth, double scale, double* __restrict__ out) {
  const int t = threadIdx.x & 63;
  const int mask = (1 << depth) - 1;
  const int i = t0 + t;
  const bool act = i < v1;
  const int li = leafid[act ? i : v0];
  const int ix = li >> depth, iy = li & mask;
  double zx = 0.0, zy = 0.0, ux = 0.0, uy = 0.0;
  bool any = false;  // the table and the targets are there
  for (int c0 = v0; c0 < v1; c0 += kOwnChunk) {
    const int cnt = min(kOwnChunk, v1 - c0);
    const int leaf = leafid[c0 + min(t, cnt - 1)];
    const int before = __shfl_up(leaf, 1);
    const bool head = t < cnt && (t == 0 || leaf != before);
    const unsigned long long hm = __ballot(head);
    const int nrun = __popcll(hm);
    wave_sync();  // the previous chunk is done
    if (head) {
      const int at = __popcll(hm & ((1ull << t) - 1ull));
      m.run0[at] = t;
      m.runl[at] = leaf;
    }
    if (t == 0) m.run0[nrun] = cnt;
    wave_sync();
    int nf = 0, ns = 0, end = -1, begin = 0;  // far points and stretches; the open stretch
    for (int r = 0; r < nrun; ++r) {
      const int lr = m.runl[r], b = m.run0[r], e = m.run0[r + 1];
      if (abs((lr >> depth) - ix) <= 1 && abs((lr & mask) - iy) <= 1) continue;
      nf += e - b;
      if (b != end) {
        if (end > 0) m.lst[ns++][t] = (uint16_t)(begin | end << 8);
        begin = b;
      }
      end = e;
    }
    if (end > 0) m.lst[ns++][t] = (uint16_t)(begin | end << 8);
    if (!act) nf = 0;
    if (!__any(nf > 0)) continue;
    if (!any) {
      m.ltab[t] = log_tab_entry(t);
      const int ii = act ? i : v0;
      zx = X[ii];
      zy = X[P + ii];
      any = true;
    }
    if (t < cnt) {
      const int j = c0 + t;
      m.sx[t] = X[j];
      m.sy[t] = X[P + j];
      m.sfx[t] = w[j] * f[j];
      m.sfy[t] = w[j] * f[P + j];
    }
    wave_sync();
    int most = nf;  // longest list of the wavefront
    for (int o = 32; o > 0; o >>= 1) most = max(most, __shfl_xor(most, o));
    int q = 0, qe = 0, s = 0;
    for (int k = 0; k < most; ++k) {
      if (k < nf) {
        if (q == qe) {
          const int se = m.lst[s++][t];
          q = se & 255;
          qe = se >> 8;
        }
        direct_term(zx, zy, m.sx[q], m.sy[q], m.sfx[q], m.sfy[q], m.ltab, ux, uy);
        ++q;
      }
    }
  }
  if (act && any) {
    out[i] = -(ux * scale);
    out[P + i] = -(uy * scale);
  }
}

// The treecode's last form of a box's rows, once the box is translated to its parent: row 3 = M_k[F] / k (k >= 1) for
// the log series of F, and row 2 = D_k, the coefficients of t^(k+1) in (S[conj F] - Psi) / 2:
// D_k = (M_{k+1}[conj F] / (k+1) - M_k[conj(zeta) F]) / 2, D_p = -M_p[conj(zeta) F] / 2.  The evaluation then needs three
// series instead of four.  Lane k brings row entries k; every lane of the wavefront takes part.
__device__ __forceinline__ void finish_box(double2* __restrict__ mb, double2 m0, double2 m1, double2 m2, int p, int k) {
  const double2 b = make_double2(__shfl_down(m1.x, 1), __shfl_down(m1.y, 1));
  asm volatile("" : "+v"(k));  // the reciprocals are formed here: kept across a caller's loop they spill
  if (k > p) return;
  double2 d = make_double2(-0.5 * m2.x, -0.5 * m2.y);
  if (k < p) {
    const double ik = 0.5 / (double)(k + 1);
    d.x = fma(b.x, ik, d.x);
    d.y = fma(b.y, ik, d.y);
  }
  mb[2 * (p + 1) + k] = d;
  mb[3 * (p + 1) + k] = k == 0 ? make_double2(0.0, 0.0) : make_double2(m0.x / (double)k, m0.y / (double)k);
}

// The same for a box whose rows are in memory.
__device__ __forceinline__ void finish_stored_box(double2* __restrict__ mb, int p, int k) {
  const int at = min(k, p);
  finish_box(mb, mb[at], mb[p + 1 + at], mb[2 * (p + 1) + at], p, k);
}

// Moments of the leaves, and of their parents where pmom is given: one workgroup per parent box, a wavefront per leaf.
// The workgroups after the nleaf / 4 of the moments form the own-vesicle terms, two wavefronts per vesicle: as a launch
// of its own that pass took 21 us at 2000 x 128 (here 17 more than the moments alone) and its start and end another
// 2 to 4; whole calls 343.5 -> 340.7 us there, near step of 2000 x 32 386.3 -> 381.8.
// A leaf's points go eight at a time: lane (b, g) = (lane mod 8, lane / 8) takes point g and the K consecutive orders
// K b .. K b + K - 1 of the 8 K >= p + 1, whose first power it forms from zeta^K in three select-multiplies, and adds
// the products of Re zeta^k and Im zeta^k with (F_x, F_y) and conj(zeta) F = (G_x, G_y) to its eight real sums per
// order.  At the end the groups' sums are exchanged so that each lane keeps one of the eight sums of its orders.
// Everything stays in registers: about 80 float64 instructions for K = 4 on eight points and 32 orders.
// 2000 x 128, order 30: this and the coarser levels 69 -> 37 us (before: powers by 32 lanes through LDS, three LDS
// reads per point and order; a launch per level whose binomials and powers were serial chains).
template <int K>
__global__ __launch_bounds__(256, K <= 4 ? 4 : 2) void k_tc_p2m(const double4* __restrict__ srec, const int32_t* __restrict__ starts,
                                                const Geom* __restrict__ geom, int depth, int p,
                                                double2* __restrict__ mom, int32_t* __restrict__ bcount,
                                                double2* __restrict__ pmom, int32_t* __restrict__ pcount, bool finish,
                                                const double* __restrict__ X, const double* __restrict__ f,
                                                const double* __restrict__ w, int P, const int32_t* __restrict__ off, int M,
                                                const int32_t* __restrict__ leafid, double scale,
                                                double* __restrict__ out) {
  struct MomentLds {
    double sums[4][8][8 * K];  // each wavefront's eight sums; then its operands and translated rows
    double2 pw[4][8 * K];
    int32_t cnt[4];
  };
  __shared__ union Lds {
    MomentLds moments;
    OwnLds own[4];
    __device__ Lds() {}
  } lds;
  auto& sums = lds.moments.sums;
  auto& pw = lds.moments.pw;
  auto& cnt = lds.moments.cnt;
  static_assert(Recentre<K>::kLds == 8 * 8 * K, "the sums and the operands share LDS");
  const int q = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
  const int own = (int)blockIdx.x - (1 << (2 * depth - 2));
  if (own >= 0) {
    const int v = 2 * own + (q >> 1);
    if (v >= M) return;
    const int v0 = clamp_i(off[v], 0, P), v1 = max(v0, clamp_i(off[v + 1], 0, P));  // offsets never trusted
    for (int t0 = v0 + 64 * (q & 1); t0 < v1; t0 += 128)
      own_terms(lds.own[q], X, f, w, P, v0, v1, t0, leafid, depth, scale, out);
    return;
  }
  const int b = lane & 7, g = lane >> 3;
  const int n = 1 << depth, box = blockIdx.x;
  const int lx = 2 * (box >> (depth - 1)) + (q >> 1), ly = 2 * (box & (n / 2 - 1)) + (q & 1);
  const int leaf = lx * n + ly;
  const int s0 = starts[leaf], s1 = starts[leaf + 1];
  const double2 c = box_center(*geom, n, lx, ly);
  const double half = 0.5 * (geom->side / (double)n);  // d = half (+-1, +-1)
  const double delta = half * 1.41421356237309504880;
  const int turn = child_turn(q);
  if (lane < 8 * K) pw[q][lane] = Recentre<K>::power(delta, turn, lane);
  double acc[K][8];
#pragma unroll
  for (int i = 0; i < K; ++i)
#pragma unroll
    for (int e = 0; e < 8; ++e) acc[i][e] = 0.0;
  double4 next = s0 < s1 ? srec[min(s0 + g, s1 - 1)] : make_double4(0.0, 0.0, 0.0, 0.0);
  for (int c0 = s0; c0 < s1; c0 += 8) {
    const double4 r = next;
    const bool ok = c0 + g < s1;
    next = srec[min(c0 + 8 + g, s1 - 1)];
    const double2 z = ok ? make_double2(r.x - c.x, r.y - c.y) : make_double2(0.0, 0.0);
    const double fx = ok ? r.z : 0.0, fy = ok ? r.w : 0.0;
    const double f4[4] = {fx, fy, fma(z.x, fx, z.y * fy), fma(z.x, fy, -(z.y * fx))};
    double2 zk = K & 1 ? z : make_double2(1.0, 0.0), sq = z;  // zeta^K
#pragma unroll
    for (int i = 2; i <= K; i <<= 1) {
      sq = cmul(sq, sq);
      if (K & i) zk = (K & (i - 1)) ? cmul(zk, sq) : sq;
    }
    double2 t = (b & 1) ? zk : make_double2(1.0, 0.0);
    zk = cmul(zk, zk);
    double2 u = cmul(t, zk);
    if (b & 2) t = u;
    zk = cmul(zk, zk);
    u = cmul(t, zk);
    if (b & 4) t = u;
#pragma unroll
    for (int i = 0; i < K; ++i) {
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        acc[i][2 * e] = fma(f4[e], t.x, acc[i][2 * e]);
        acc[i][2 * e + 1] = fma(f4[e], t.y, acc[i][2 * e + 1]);
      }
      if (i + 1 < K) t = cmul(t, z);
    }
  }
  const Recentre<K> up(p);  // its operand loads while the sums are exchanged
  // the groups' sums: each exchange halves the sums a lane keeps
#pragma unroll
  for (int i = 0; i < K; ++i) {
    double* a = acc[i];
#pragma unroll
    for (int e = 0; e < 4; ++e) a[e] = pair_sums<32>(a[e], a[e + 4], lane);
#pragma unroll
    for (int e = 0; e < 2; ++e) a[e] = pair_sums<16>(a[e], a[e + 2], lane);
    sums[q][g][K * b + i] = pair_sums<8>(a[0], a[1], lane);
  }
  wave_sync();
  double2 m0 = make_double2(0.0, 0.0), m1 = m0, m2 = m0;
  if (lane <= p) {
    const auto S = [&](int e) { return sums[q][e][lane]; };  // sums of (F_x, F_y, G_x, G_y) times (Re, Im)
    m0 = make_double2(S(0) - S(3), S(1) + S(2));
    m1 = make_double2(S(0) + S(3), S(1) - S(2));
    m2 = make_double2(S(4) - S(7), S(5) + S(6));
    double2* mb = mom + (size_t)leaf * 4 * (p + 1);
    mb[lane] = m0;
    mb[p + 1 + lane] = m1;
    if (!finish) mb[2 * (p + 1) + lane] = m2;
  }
  if (finish) finish_box(mom + (size_t)leaf * 4 * (p + 1), m0, m1, m2, p, lane);
  if (lane == 0) bcount[leaf] = cnt[q] = s1 - s0;
  if (pmom == nullptr) return;
  wave_sync();
  up.run(m0, m1, m2, delta, turn, pw[q], &sums[q][0][0]);
  __syncthreads();
  double2* pm = pmom + (size_t)box * 4 * (p + 1);
  for (int e = threadIdx.x; e < 3 * (p + 1); e += 256) pm[e] = children_sum(&sums[0][0][0], Recentre<K>::kLds, p, half, e);
  if (threadIdx.x == 0) pcount[box] = cnt[0] + cnt[1] + cnt[2] + cnt[3];
  if (finish && depth == 3) {  // the parents are the coarsest boxes
    __syncthreads();
    if (q == 0) finish_stored_box(pm, p, lane);
  }
}

// Moments of the levels from `from` up to `to` (from >= to >= 2) from those of level from + 1: one workgroup per box of
// level `to` works through its boxes of every level, a wavefront per child, four for a box, which also brings the child
// to the treecode's last form where `finish` is given (as a launch of its own that took 5 us).  Latency bounds it, about
// 3 us for sixteen children.
constexpr int up_waves(int K) { return K < 7 ? 16 : 8; }  // K = 7 needs more than 128 registers

template <int K>
__global__ __launch_bounds__(64 * up_waves(K)) void k_tc_m2m(const Geom* __restrict__ geom, int from, int to, int p,
                                                          double2* __restrict__ mom, int32_t* __restrict__ bcount,
                                                          bool finish) {
  __shared__ double x[up_waves(K)][Recentre<K>::kLds];
  __shared__ double2 pw[4][8 * K];
  __shared__ int32_t cnt[up_waves(K)];
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), boxes = blockDim.x >> 8, lane = threadIdx.x & 63;
  const int q = wave & 3;
  const int tx = blockIdx.x >> to, ty = blockIdx.x & ((1 << to) - 1);
  const int stride = 4 * (p + 1), used = 3 * (p + 1);
  const double side = geom->side;
  const int turn = child_turn(q);
  const Recentre<K> up(p);
  for (int l = from; l >= to; --l) {
    const double half = 0.5 * (side / (double)(2 << l));  // of a child's width
    const double delta = half * 1.41421356237309504880;
    const int sh = l - to;
    if (wave < 4 && lane < 8 * K) pw[wave][lane] = Recentre<K>::power(delta, turn, lane);
    __syncthreads();
    for (int i0 = 0; i0 < 1 << (2 * sh); i0 += boxes) {
      const int i = i0 + (wave >> 2);
      if (i < 1 << (2 * sh)) {
        const int bx = (tx << sh) + (i >> sh), by = (ty << sh) + (i & ((1 << sh) - 1));
        const size_t cb = level_box_base(l + 1) + ((size_t)(2 * bx + (q >> 1)) << (l + 1)) + (2 * by + (q & 1));
        double2 m0 = make_double2(0.0, 0.0), m1 = m0, m2 = m0;
        if (lane <= p) {
          const double2* mb = mom + cb * stride;
          m0 = mb[lane];
          m1 = mb[p + 1 + lane];
          m2 = mb[2 * (p + 1) + lane];
        }
        if (finish) finish_box(mom + cb * stride, m0, m1, m2, p, lane);
        if (lane == 0) cnt[wave] = bcount[cb];
        up.run(m0, m1, m2, delta, turn, pw[q], x[wave]);
      }
      __syncthreads();
      const int mine = min(boxes, (1 << (2 * sh)) - i0);
      for (int e = threadIdx.x; e < mine * used; e += blockDim.x) {
        const int c = e / used, k = e - c * used, ib = i0 + c;
        const int bx = (tx << sh) + (ib >> sh), by = (ty << sh) + (ib & ((1 << sh) - 1));
        const size_t box = level_box_base(l) + ((size_t)bx << l) + by;
        mom[box * stride + k] = children_sum(x[4 * c], Recentre<K>::kLds, p, half, k);
        if (k == 0) bcount[box] = cnt[4 * c] + cnt[4 * c + 1] + cnt[4 * c + 2] + cnt[4 * c + 3];
      }
      __syncthreads();  // LDS is free, and this level's boxes are written
    }
  }
  if (finish && to == 2 && wave == 0)  // no level above: this workgroup's box is finished here
    finish_stored_box(mom + (level_box_base(2) + blockIdx.x) * stride, p, lane);
}

// ---------------------------------------------------------------- fast multipole translations
//
// Local expansion of a box T (centre c_T, zeta = z - c_T): three rows of (p + 1) complex Taylor
// coefficients A, B, C such that the far field (times 4 pi mu) of everything in the interaction lists
// of T and of its ancestors is
//     u = -A(zeta)/2 - conj(B(zeta))/2 + zeta conj(C(zeta))/2.
// A source box S, d = c_S - c_T, t = 1/d, enters through its multipole series in powers of (z - c_S)^-1:
//   A: log sum of F,  lambda = M_0[F],       a_m = -M_m[F]/m                      (m = 1..p);
//   C: Cauchy sum Phi,                       a_m = M_{m-1}[F]                     (m = 1..p+1);
//   B: log sum of conj F plus Psi,  lambda = M_0[conj F],  a_m = -M_m[conj F]/m + M_{m-1}[conj(zeta) F],
//      plus conj(d) times C (the term that re-centres conj(zeta_j) from c_S to c_T).
// With (z - c_S)^-m = (-t)^m sum_l C(m + l - 1, l) t^l zeta^l and log(z - c_S) = log(-d) - sum_{l>=1} t^l zeta^l / l,
// the coefficient of zeta^l is t^l (sum_m C(m + l - 1, l) (-t)^m a_m - lambda / l), and for l = 0
// lambda ln|d| + sum_m (-t)^m a_m: the imaginary part of log(-d) cancels between A and conj(B) because
// M_0[conj F] = conj(M_0[F]).  Each source box's constant M_0[F]/2 goes into A_0 as -M_0[F].
// A child inherits its parent's expansion re-centred by e = c_child - c_parent:
//   X_l += sum_{m>=l} C(m, l) e^(m-l) X_m  for A, B, C, and B additionally -conj(e) times the shifted C.

// Dynamic LDS of k_fmm_m2l for order p, KS = ceil((p + 1) / 4) steps of four m and RT = ceil((p + 1) / 16)
// tiles of 16 orders: the source list, the scaled coefficients
// X[v][m - 1][s] of a batch (3 series x 4 KS x 8 sources, complex; also the final exchange of 3 x 64 sums),
// the powers (-t_s)^l (8 sources x 4 KS, complex), and per source lambda_A, lambda_B (complex) and ln|d|.
// (Splitting a box's batches over several waves, or taking one series at a time to save registers, both
// measured slower: the first is limited by LDS occupancy, the second loses independent MFMA chains.)
constexpr int kM2LBatch = 8;  // source boxes per batch: 8 complex columns fill one 16-column tile
__host__ __device__ inline int m2l_ksteps(int p) { return (p + 1 + 3) / 4; }
__host__ __device__ inline int m2l_rtiles(int p) { return (p + 1 + 15) / 16; }
__host__ __device__ inline int m2l_xsize(int p) {  // in double2
  const int mm = 4 * m2l_ksteps(p);
  return 3 * mm * kM2LBatch > 3 * 64 ? 3 * mm * kM2LBatch : 3 * 64;
}
inline size_t m2l_lds_bytes(int p) {
  const int mm = 4 * m2l_ksteps(p);
  return sizeof(double2) * ((size_t)36 + m2l_xsize(p) + (size_t)kM2LBatch * mm + 2 * kM2LBatch +
                            kM2LBatch / 2);
}

// 1 / (m + 1), m = 0..kMaxOrder.
__constant__ double kRecip[kMaxOrder + 1] = {
    1.0 / 1,  1.0 / 2,  1.0 / 3,  1.0 / 4,  1.0 / 5,  1.0 / 6,  1.0 / 7,  1.0 / 8,  1.0 / 9,  1.0 / 10,
    1.0 / 11, 1.0 / 12, 1.0 / 13, 1.0 / 14, 1.0 / 15, 1.0 / 16, 1.0 / 17, 1.0 / 18, 1.0 / 19, 1.0 / 20,
    1.0 / 21, 1.0 / 22, 1.0 / 23, 1.0 / 24, 1.0 / 25, 1.0 / 26, 1.0 / 27, 1.0 / 28, 1.0 / 29, 1.0 / 30,
    1.0 / 31, 1.0 / 32, 1.0 / 33, 1.0 / 34, 1.0 / 35, 1.0 / 36, 1.0 / 37, 1.0 / 38, 1.0 / 39, 1.0 / 40,
    1.0 / 41, 1.0 / 42, 1.0 / 43, 1.0 / 44, 1.0 / 45, 1.0 / 46, 1.0 / 47, 1.0 / 48, 1.0 / 49};

// Interaction-list contributions to the local expansion of every non-empty box of levels 2..depth (one
// launch for all levels, one wavefront per target box), on the matrix cores.  For a source box s at
// d_s = c_s - c_T, t_s = 1/d_s, and each series v (A, Phi, and B with the conj(d) Phi term folded in,
// conj(d_s) being a constant factor per source), the coefficient of zeta^l is
//   t_s^l (sum_{m=1}^{p+1} C(m + l - 1, l) X_v[m][s] - lambda_v / l),   X_v[m][s] = a_v(m) (-t_s)^m,
// (l = 0: sum_m X_v[m][s] + lambda_v ln|d_s|).  The sums over m are the product D = X^T T with
// X^T: (16 columns: 8 sources x re, im) x m and T: m x l, in 16 x 16 x 4 FP64 steps: the columns of a tile
// are one series of eight sources, source c's real part in row (c mod 4) + 8 (c / 4) and its imaginary part
// four rows below, so that every lane (l = lane mod 16, q = lane / 16) receives both parts of sources q and
// q + 4 for its order l and scales them itself.  Sources go eight at a time, in the fixed candidate order;
// at the end the sums of the four lanes of every order are added in q order.  RT = ceil((p + 1) / 16).
// At least two wavefronts per SIMD: with 256 VGPRs at most the compiler keeps D in VGPRs, where the matrix
// instructions can add to it; with more it copied all of D to accumulation registers and back at every step (96 of
// its 125 instructions).  The binomials come from L1 one step ahead: staged in LDS they were a third of the LDS that
// held the kernel to six wavefronts per CU.  2000 x 128, order 30: 124 -> 84 us.  (48 orders need more registers.)
template <int RT>
__global__ __launch_bounds__(64, RT < 4 ? 2 : 1) void k_fmm_m2l(const Geom* __restrict__ geom, int depth, int p,
                                                           const double2* __restrict__ mom,
                                                           const int32_t* __restrict__ bcount,
                                                           double2* __restrict__ loc) {
  extern __shared__ double2 sm[];
  const size_t box = blockIdx.x;
  if (bcount[box] == 0) return;
  const int lane = threadIdx.x;
  const int np = p + 1;
  const int KS = m2l_ksteps(p), MM = 4 * KS;
  int32_t* lst = reinterpret_cast<int32_t*>(sm);                 // [36][2]: source box coordinates
  double2* X = sm + 36;                                          // [3][MM][8]
  double2* pw = X + m2l_xsize(p);                                // [8][MM]: (-t_s)^l
  double2* lam = pw + kM2LBatch * MM;                            // [8][2]: lambda_A, lambda_B
  double* lnd = reinterpret_cast<double*>(lam + 2 * kM2LBatch);  // [8]
  int l2 = 2;
  while (l2 < depth && box >= level_box_base(l2 + 1)) ++l2;
  const int n = 1 << l2;
  const size_t base = level_box_base(l2);
  const int b = (int)(box - base);
  const int bx = b / n, by = b - (b / n) * n;
  const double wl = geom->side / (double)n;
  const int stride = 4 * np;
  // the interaction list's non-empty boxes in the fixed candidate order: lane c examines candidate c
  int ns;
  {
    const int sx = 2 * (bx >> 1) + lane / 6 - 2, sy = 2 * (by >> 1) + lane % 6 - 2;
    bool ok = lane < 36 && sx >= 0 && sx < n && sy >= 0 && sy < n && (abs(sx - bx) > 1 || abs(sy - by) > 1);
    if (ok) ok = bcount[base + (size_t)sx * n + sy] != 0;
    const unsigned long long mask = __ballot(ok);
    ns = __popcll(mask);
    if (ok) {
      const int rank = __popcll(mask & ((1ull << lane) - 1ull));
      lst[2 * rank] = sx;
      lst[2 * rank + 1] = sy;
    }
  }
  wave_sync();  // list ready
  const int j = lane & 15, q = lane >> 4;  // result lanes: order j (+ 16 rt), sources q and q + 4
  const int ai = lane & 15, ak = lane >> 4;  // operand lanes: column / order ai, step row ak
  const int acol = (ai & 3) + 4 * (ai >> 3), apart = (ai >> 2) & 1;  // column ai: source acol, re or im
  double2 acc[3][RT];
  double inv_l[RT];  // 1/l for the lane's orders l = j + 16 rt (0 for l = 0 or beyond p)
#pragma unroll
  for (int rt = 0; rt < RT; ++rt) {
    const int l = j + 16 * rt;
    inv_l[rt] = (l >= 1 && l <= p) ? kRecip[l - 1] : 0.0;
#pragma unroll
    for (int v = 0; v < 3; ++v) acc[v][rt] = make_double2(0.0, 0.0);
  }
  for (int b0 = 0; b0 < ns; b0 += kM2LBatch) {
    const int nb = min(kM2LBatch, ns - b0);
    // scaling: lane takes source s = lane mod 8 and m = 1 + lane / 8, then every eighth m
    {
      const int s = lane & 7;
      const bool valid = s < nb;
      const int sx = valid ? lst[2 * (b0 + s)] : bx + 2, sy = valid ? lst[2 * (b0 + s) + 1] : by;
      const double2 d = make_double2((double)(sx - bx) * wl, (double)(sy - by) * wl);
      const double dd = d.x * d.x + d.y * d.y;
      const double rdd = recip(dd);
      const double2 mt = make_double2(-d.x * rdd, d.y * rdd);  // -t
      const double2* ms = mom + (base + (size_t)(valid ? sx : 0) * n + (valid ? sy : 0)) * stride;
      const int m0 = 1 + (lane >> 3);
      // every moment load first, at indices clamped into the rows (values outside are discarded), so
      // that they are all in flight together
      double2 Fm1[2 * RT], Fm[2 * RT], Cm[2 * RT], Pm1[2 * RT];
#pragma unroll
      for (int it = 0; it < 2 * RT; ++it) {
        const int mc = min(m0 + 8 * it, np), mp = min(mc, p);
        Fm1[it] = ms[mc - 1];
        Fm[it] = ms[mp];
        Cm[it] = ms[np + mp];
        Pm1[it] = ms[2 * np + mc - 1];
      }
      const double2 t2 = cmul(mt, mt), t4 = cmul(t2, t2), step = cmul(t4, t4);  // (-t)^2, ^4, ^8
      const int e0 = m0 - 1;                                                     // 0..7
      double2 pl = (e0 & 1) ? mt : make_double2(1.0, 0.0);                      // (-t)^(m-1)
      if (e0 & 2) pl = cmul(pl, t2);
      if (e0 & 4) pl = cmul(pl, t4);
#pragma unroll
      for (int it = 0; it < 2 * RT; ++it) {  // m = m0 + 8 it; MM <= 16 RT
        const int m = m0 + 8 * it;
        if (m <= MM) {
          pw[s * MM + (m - 1)] = valid ? pl : make_double2(0.0, 0.0);
          const bool use = valid && m <= np;
          const double2 pm = cmul(pl, mt);  // (-t)^m
          const double im = m <= p ? kRecip[m - 1] : 0.0;  // the A and conj-F series stop at order p
          const double2 aA = make_double2(-Fm[it].x * im, -Fm[it].y * im);
          const double2 aQ = make_double2(fma(-Cm[it].x, im, Pm1[it].x), fma(-Cm[it].y, im, Pm1[it].y));
          const double2 sh = cmul(make_double2(d.x, -d.y), Fm1[it]);  // conj(d) Phi folded into B
          const double2 zero = make_double2(0.0, 0.0);
          X[(0 * MM + (m - 1)) * kM2LBatch + s] = use ? cmul(aA, pm) : zero;
          X[(1 * MM + (m - 1)) * kM2LBatch + s] = use ? cmul(Fm1[it], pm) : zero;
          X[(2 * MM + (m - 1)) * kM2LBatch + s] = use ? cmul(make_double2(aQ.x + sh.x, aQ.y + sh.y), pm) : zero;
        }
        pl = cmul(pl, step);
      }
      if (lane < kM2LBatch) {  // lane = s, m0 = 1: the first load of the loop above read M_0[F]
        const double2 lq = ms[np];
        lam[2 * s] = valid ? Fm1[0] : make_double2(0.0, 0.0);
        lam[2 * s + 1] = valid ? lq : make_double2(0.0, 0.0);
        lnd[s] = valid ? 0.5 * log_pos(dd) : 0.0;
      }
    }
    wave_sync();
    // D[v][rt] = sum over m of the batch's columns times the binomials, three series and RT order tiles
    // issued together at every step
    const double* Xd = reinterpret_cast<const double*>(X);
    double4v D[3][RT];
#pragma unroll
    for (int v = 0; v < 3; ++v)
#pragma unroll
      for (int rt = 0; rt < RT; ++rt) D[v][rt] = (double4v){0.0, 0.0, 0.0, 0.0};
    double bn[RT];  // the next step's binomials, loaded one step ahead
#pragma unroll
    for (int rt = 0; rt < RT; ++rt) bn[rt] = kBinomials.t[ak][ai + 16 * rt];
    for (int ks = 0; ks < KS; ++ks) {
      const int mi = 4 * ks + ak, mn = 4 * min(ks + 1, KS - 1) + ak;  // m - 1, and the next step's
      double av[3], bv[RT];
#pragma unroll
      for (int v = 0; v < 3; ++v) av[v] = Xd[2 * ((v * MM + mi) * kM2LBatch + acol) + apart];
#pragma unroll
      for (int rt = 0; rt < RT; ++rt) {
        bv[rt] = bn[rt];
        bn[rt] = kBinomials.t[mn][ai + 16 * rt];
      }
#pragma unroll
      for (int v = 0; v < 3; ++v)
#pragma unroll
        for (int rt = 0; rt < RT; ++rt) D[v][rt] = __builtin_amdgcn_mfma_f64_16x16x4f64(av[v], bv[rt], D[v][rt], 0, 0, 0);
    }
    // scale: every lane owns orders l = j + 16 rt and sources q, q + 4; t^l, 1/l, the lambdas and ln|d|
    // are shared by the three series
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const int s = q + 4 * h;
      const double2 lamA = lam[2 * s], lamB = lam[2 * s + 1];
      const double ld = lnd[s];
#pragma unroll
      for (int rt = 0; rt < RT; ++rt) {
        const int l = j + 16 * rt;
        if (l > p) continue;
        const double2 pwl = pw[s * MM + l];
        const double sg = (l & 1) ? -1.0 : 1.0;  // t^l = (-1)^l (-t)^l
        const double2 tl = l == 0 ? make_double2(1.0, 0.0) : make_double2(sg * pwl.x, sg * pwl.y);
        const double il = inv_l[rt];
#pragma unroll
        for (int v = 0; v < 3; ++v) {
          const double2 y = make_double2(D[v][rt][2 * h], D[v][rt][2 * h + 1]);
          const double2 lv = v == 0 ? lamA : (v == 2 ? lamB : make_double2(0.0, 0.0));
          // l = 0: y + lambda ln|d| (and, for A, the source's constant M_0[F] / 2 as -M_0[F]);
          // l >= 1: t^l (y - lambda / l)
          const double2 c0 = make_double2(fma(lv.x, l == 0 ? ld : -il, y.x), fma(lv.y, l == 0 ? ld : -il, y.y));
          double2 bv2 = cmul(tl, c0);
          if (v == 0 && l == 0) {
            bv2.x -= lv.x;
            bv2.y -= lv.y;
          }
          acc[v][rt].x += bv2.x;
          acc[v][rt].y += bv2.y;
        }
      }
    }
    wave_sync();  // the staging is rewritten by the next batch
  }
  // the sums of the four lanes of every order, added in q order; X is reused for the exchange
  double2* lb = loc + box * 3 * np;
#pragma unroll
  for (int rt = 0; rt < RT; ++rt) {
#pragma unroll
    for (int v = 0; v < 3; ++v) X[v * 64 + lane] = acc[v][rt];
    wave_sync();
    const int l = lane + 16 * rt;
    if (lane < 16 && l <= p) {
      for (int v = 0; v < 3; ++v) {
        double2 r = X[v * 64 + lane];
        for (int qq = 1; qq < 4; ++qq) {
          r.x += X[v * 64 + lane + 16 * qq].x;
          r.y += X[v * 64 + lane + 16 * qq].y;
        }
        lb[(v == 0 ? 0 : (v == 1 ? 2 : 1)) * np + l] = r;  // series A, Phi, B -> rows A, B, C
      }
    }
    wave_sync();
  }
}

// Completes the local expansion of every non-empty leaf: its own interaction-list part plus the part of
// each ancestor (levels 2..depth-1), re-centred from the ancestor's centre straight to the leaf's (the
// re-centring of a polynomial is exact, so one shift per ancestor equals the chain through the levels).
// With e = c_leaf - c_anc: X_k += sum_{m>=k} C(m, k) e^(m-k) X_m for A, B, C, and B also -conj(e) times the
// shifted C.  One wavefront per leaf, on the matrix cores: X_k = e^-k sum_m C(m, k) (e^m X_m), the triangle of binomials
// the first operand (in registers, shared by all ancestors) and the e^m X_m of two ancestors, six real columns each,
// the second.  For 8 K >= p + 1 orders.  Powers of e are real powers of |e| times powers of e / |e|; the power of two of
// |e| is taken apart and scales exactly, the rest lies in [1/2, 1), so that no power overflows (the orders above p hold
// zeros, and zero times infinity would spoil every order).
// 2000 x 128, order 30: 25 -> 16.7 us (before: a lane per order, binomials and powers serial chains, three LDS reads
// per term).
constexpr int kShiftWaves = 4;

template <int K>
__global__ __launch_bounds__(64 * kShiftWaves) void k_fmm_l2l(const Geom* __restrict__ geom, int depth, int p,
                                                              const int32_t* __restrict__ bcount,
                                                              double2* __restrict__ loc) {
  constexpr int kTiles = (K + 1) / 2, kOrders = 8 * K;
  constexpr int kRow = 17;  // doubles per order: 16 columns and a spare one against bank conflicts
  __shared__ double xs[kShiftWaves][kOrders * kRow + 1];
  __shared__ double2 inv[kShiftWaves][2][kOrders];
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
  const int n = 1 << depth;
  const int leaf = blockIdx.x * kShiftWaves + wave;
  const size_t lbox = level_box_base(depth) + (size_t)leaf;
  if (bcount[lbox] == 0) return;
  double* x = xs[wave];
  const int bx = leaf / n, by = leaf % n;
  const int rows = 3 * (p + 1);
  const double wL = geom->side / (double)n;
  double a[kTiles][2 * K];
#pragma unroll
  for (int rt = 0; rt < kTiles; ++rt)
#pragma unroll
    for (int s = 4 * rt; s < 2 * K; ++s) {
      const int k = 16 * rt + (lane & 15), m = 4 * s + (lane >> 4);
      const double c = kBinomials.t[min(k, kTabM - 1)][max(m - k, 0)];  // C(m, k)
      a[rt][s] = m >= k ? c : 0.0;
    }
  const int c = lane & 15, series = (c & 7) >> 1;
  double tot[kTiles][4];
#pragma unroll
  for (int rt = 0; rt < kTiles; ++rt)
#pragma unroll
    for (int v = 0; v < 4; ++v) tot[rt][v] = 0.0;
  for (int l0 = 2; l0 < depth; l0 += 2) {
    double2 e[2];
    int ex[2];  // |e| = (1/2 .. 1) 2^ex
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const int l = l0 + h, sh = depth - l;
      const int ax = bx >> sh, ay = by >> sh;
      // leaf centre - ancestor centre = ((b + 1/2) - (a + 1/2) 2^sh) wL per coordinate: exact before the product
      e[h] = make_double2(((double)bx + 0.5 - ((double)ax + 0.5) * (double)(1 << sh)) * wL,
                          ((double)by + 0.5 - ((double)ay + 0.5) * (double)(1 << sh)) * wL);
      double2 v[3] = {make_double2(0.0, 0.0), make_double2(0.0, 0.0), make_double2(0.0, 0.0)};
      if (l < depth && lane <= p) {
        const double2* pa = loc + (level_box_base(l) + ((size_t)ax << l) + ay) * rows + lane;
        v[0] = pa[0];
        v[1] = pa[p + 1];
        v[2] = pa[2 * (p + 1)];
      }
      if (l == depth) e[h] = make_double2(1.0, 0.0);  // no ancestor: zero columns
      const double r = sqrt(e[h].x * e[h].x + e[h].y * e[h].y), ri = 1.0 / r;
      const double rf = frexp(r, &ex[h]);
      if (lane < kOrders) {
        const double2 u = cpow_int(make_double2(e[h].x * ri, e[h].y * ri), lane);
        const double rm = pow_int(rf, lane), rk = pow_int(1.0 / rf, lane);
        inv[wave][h][lane] = make_double2(u.x * rk, -(u.y * rk));
        const double2 em = make_double2(u.x * rm, u.y * rm);
#pragma unroll
        for (int q = 0; q < 3; ++q) {
          const double2 t = cmul(make_double2(ldexp(v[q].x, ex[h] * lane), ldexp(v[q].y, ex[h] * lane)), em);
          x[kRow * lane + 8 * h + 2 * q] = t.x;
          x[kRow * lane + 8 * h + 2 * q + 1] = t.y;
        }
      }
    }
    wave_sync();
    double4v acc[kTiles];
#pragma unroll
    for (int rt = 0; rt < kTiles; ++rt) acc[rt] = double4v{0.0, 0.0, 0.0, 0.0};
#pragma unroll
    for (int s = 0; s < 2 * K; ++s) {
      const double b = x[kRow * (4 * s + (lane >> 4)) + c];
#pragma unroll
      for (int rt = 0; rt < kTiles; ++rt)
        if (s >= 4 * rt) acc[rt] = __builtin_amdgcn_mfma_f64_16x16x4f64(a[rt][s], b, acc[rt], 0, 0, 0);
    }
    const double2 eh = (c & 8) ? e[1] : e[0];
    const int exh = (c & 8) ? ex[1] : ex[0];
#pragma unroll
    for (int rt = 0; rt < kTiles; ++rt)
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const int k = 16 * rt + (lane >> 4) + 4 * v;
        const double2 ik = inv[wave][c >> 3][min(k, kOrders - 1)];
        const double mine = acc[rt][v], other = quad_swap(mine);  // Re and Im are neighbours
        const double val = ldexp(fma(mine, ik.x, (c & 1) ? other * ik.y : -(other * ik.y)), -exh * k);
        const double cm = row_shift2(val), co = quad_swap(cm);  // for the lanes of B: C and its other part
        const double shc = fma(eh.x, cm, (c & 1) ? -(eh.y * co) : eh.y * co);  // conj(e) C
        tot[rt][v] += series == 1 ? val - shc : val;
      }
    wave_sync();  // x and inv are read
  }
#pragma unroll
  for (int rt = 0; rt < kTiles; ++rt)
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const int k = 16 * rt + (lane >> 4) + 4 * v;
      const double sum = tot[rt][v] + row_half(tot[rt][v]);  // the two ancestors of a pair
      if (c < 6 && k <= p) x[2 * (series * (p + 1) + k) + (c & 1)] = sum;
    }
  wave_sync();
  double2* lb = loc + lbox * rows;
  for (int t = lane; t < rows; t += 64) {
    const double2 v = lb[t];
    lb[t] = make_double2(v.x + x[2 * t], v.y + x[2 * t + 1]);
  }
}

// ---------------------------------------------------------------- evaluation

// The leaf of a work item, wstart[leaf] <= item < wstart[leaf + 1]: 64 places are looked at together, so 4,096 leaves
// take two rounds of memory latency (a binary search took twelve).
__device__ __forceinline__ int leaf_of_item(const int32_t* __restrict__ wstart, int nleaf, int item) {
  const int lane = threadIdx.x & 63;
  int lo = 0, end = nleaf;  // wstart[lo] <= item < wstart[end]
  while (end - lo > 1) {
    const int step = (end - lo + 63) >> 6;
    const int at = lo + (lane + 1) * step;
    const int k = __popcll(__ballot(at < end && wstart[min(at, end)] <= item));
    lo += k * step;
    end = min(lo + step, end);
  }
  return lo;
}

// ---------------------------------------------------------------- fast multipole evaluation
//
// One wavefront per (leaf, chunk of 16 of its points), four to a workgroup, which share the 1024-entry log table:
// 8 lanes take two targets each and the 8 lane groups share the sources of the 3 x 3 leaves (every 8th) and the
// terms of the leaf's local expansion (group g the powers g, g + 8, ...: Horner in zeta^8, then zeta^g); the groups'
// sums are added at the end.  The three leaves of a column are one run of the leaf order, and the three runs are
// staged as one list, 64 records at a time with the next 64 loading meanwhile.  Two targets per lane use each record
// read from LDS twice.  What bounds it is float64 VALU issue, 31 instructions per (target, source).
// 2000 x 128, order 30: 263 -> 187 us (160 at one instruction per 4 cycles).
constexpr int kFmmT = 2;
constexpr int kFmmLanes = 8;
constexpr int kFmmGroups = 64 / kFmmLanes;
constexpr int kFmmChunkShift = 4;  // log2 of the targets per wavefront
constexpr int kFmmWaves = 4;       // wavefronts per workgroup
static_assert(1 << kFmmChunkShift == kFmmT * kFmmLanes, "every lane of a group takes kFmmT targets");

__global__ __launch_bounds__(64 * kFmmWaves) void k_fmm_eval(const double4* __restrict__ srec,
                                                             const int32_t* __restrict__ svid, int P,
                                                             const int32_t* __restrict__ perm,
                                                             const int32_t* __restrict__ starts,
                                                             const int32_t* __restrict__ wstart,
                                                             const Geom* __restrict__ geom, int depth, int p,
                                                             const double2* __restrict__ loc,
                                                             const double2* __restrict__ tab, double scale,
                                                             double* __restrict__ out) {
  __shared__ double2 ltab[kHalfLogTab];
  // per wavefront: 64 source records and ids, then the local expansion (3 (p + 1) <= 147 entries)
  __shared__ double2 stage[kFmmWaves][3 * 64];
  for (int e = threadIdx.x; e < kHalfLogTab; e += 64 * kFmmWaves) ltab[e] = tab[e];
  const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
  double2* cf = stage[wv];
  double4* src = reinterpret_cast<double4*>(stage[wv]);
  int32_t* sv = reinterpret_cast<int32_t*>(stage[wv] + 2 * 64);
  const int n = 1 << depth;
  const int nleaf = n * n;
  const int item = blockIdx.x * kFmmWaves + wv;
  const bool some = item < wstart[nleaf];
  const int leaf = some ? leaf_of_item(wstart, nleaf, item) : 0;
  __syncthreads();
  if (!some) return;
  const int s1 = starts[leaf + 1];
  const int base = starts[leaf] + ((item - wstart[leaf]) << kFmmChunkShift);
  const int tl = lane & (kFmmLanes - 1), grp = lane / kFmmLanes;
  const int ix = leaf / n, iy = leaf % n;
  // the source runs of columns ix - 1 .. ix + 1 (empty outside the grid), as one list of nsrc slots
  int run0[3], cum[4];
  cum[0] = 0;
#pragma unroll
  for (int a = 0; a < 3; ++a) {
    const int jx = ix + a - 1;
    const bool in = jx >= 0 && jx < n;
    run0[a] = in ? starts[jx * n + max(iy - 1, 0)] : 0;
    cum[a + 1] = cum[a] + (in ? starts[jx * n + min(iy + 1, n - 1) + 1] - run0[a] : 0);
  }
  const int nsrc = cum[3];
  auto slot_of = [&](int e) {
    return e < cum[1] ? run0[0] + e : e < cum[2] ? run0[1] + e - cum[1] : run0[2] + e - cum[2];
  };
  // nsrc >= 1: the leaf itself is in the list
  double4 nrec = srec[slot_of(min(lane, nsrc - 1))];
  int nvid = svid[slot_of(min(lane, nsrc - 1))];

  double zx[kFmmT], zy[kFmmT], ux[kFmmT], uy[kFmmT];
  int ti[kFmmT], vi[kFmmT];
#pragma unroll
  for (int k = 0; k < kFmmT; ++k) {
    const int slot = base + tl + kFmmLanes * k;
    const int sl = slot < s1 ? slot : base;  // an empty slot repeats the first target
    ti[k] = perm[sl];
    const double4 z = srec[sl];
    zx[k] = z.x;
    zy[k] = z.y;
    vi[k] = svid[sl];
    ux[k] = uy[k] = 0.0;
  }
  // the 3 x 3 leaves directly, own vesicle skipped
  for (int c0 = 0; c0 < nsrc; c0 += 64) {
    const int cnt = min(64, nsrc - c0);
    wave_sync();  // the previous records are done
    src[lane] = nrec;
    sv[lane] = nvid;
    wave_sync();
    if (c0 + 64 < nsrc) {
      const int sl = slot_of(min(c0 + 64 + lane, nsrc - 1));
      nrec = srec[sl];
      nvid = svid[sl];
    }
    for (int q = grp; q < cnt; q += kFmmGroups) {
      const double4 s = src[q];
      const int cv = sv[q];
#pragma unroll
      for (int k = 0; k < kFmmT; ++k)
        if (cv != vi[k]) {
          const double rx = zx[k] - s.x, ry = zy[k] - s.y;
          const double d2 = fma(ry, ry, rx * rx);
          const double l = neg_half_log(d2, ltab);
          const double t = fma(ry, s.w, rx * s.z) * recip(d2);
          ux[k] = fma(l, s.z, fma(t, rx, ux[k]));
          uy[k] = fma(l, s.w, fma(t, ry, uy[k]));
        }
    }
  }
  // the leaf's local expansion: u += -A(zeta)/2 - conj(B(zeta))/2 + zeta conj(C(zeta))/2, linear in the terms;
  // after the direct part, whose many terms would each round at the size of the whole (3 times the error at order 40)
  if (depth >= 2) {
    const int np = p + 1;
    const double2* lb = loc + (level_box_base(depth) + (size_t)leaf) * 3 * np;
    wave_sync();  // the records are done
#pragma unroll
    for (int u = 0; u < 3; ++u)
      if (lane + 64 * u < 3 * np) cf[lane + 64 * u] = lb[lane + 64 * u];
    wave_sync();
    const double2 c = box_center(*geom, n, ix, iy);
    const int k1 = grp + kFmmGroups * ((p - grp) / kFmmGroups);  // highest power of the group (if grp <= p)
#pragma unroll
    for (int k = 0; k < kFmmT; ++k) {
      const double2 zt = make_double2(zx[k] - c.x, zy[k] - c.y);
      const double2 z2 = cmul(zt, zt), z4 = cmul(z2, z2), z8 = cmul(z4, z4);
      double2 zg = (grp & 1) ? zt : make_double2(1.0, 0.0);
      if (grp & 2) zg = cmul(zg, z2);
      if (grp & 4) zg = cmul(zg, z4);
      double2 A = make_double2(0.0, 0.0), B = A, C = A;
      if (grp <= p)
        for (int q = k1; q >= 0; q -= kFmmGroups) {
          A = cfma(A, z8, cf[q]);
          B = cfma(B, z8, cf[np + q]);
          C = cfma(C, z8, cf[2 * np + q]);
        }
      A = cmul(A, zg);
      B = cmul(B, zg);
      C = cmul(C, zg);
      ux[k] += -0.5 * A.x - 0.5 * B.x + 0.5 * (zt.x * C.x + zt.y * C.y);
      uy[k] += -0.5 * A.y + 0.5 * B.y + 0.5 * (zt.y * C.x - zt.x * C.y);
    }
  }
#pragma unroll
  for (int k = 0; k < kFmmT; ++k) {  // the groups' sums, pairwise in a fixed order
#pragma unroll
    for (int o = kFmmLanes; o < 64; o <<= 1) {
      ux[k] += __shfl_xor(ux[k], o);
      uy[k] += __shfl_xor(uy[k], o);
    }
    if (grp == 0 && base + tl + kFmmLanes * k < s1) {
      out[ti[k]] += ux[k] * scale;  // to the own-vesicle terms
      out[P + ti[k]] += uy[k] * scale;
    }
  }
}

// ---------------------------------------------------------------- treecode evaluation
//
// One workgroup per part of a leaf of at most 32 points (a leaf's parts are of equal size), four wavefronts: L = 8 .. 16
// lanes take two targets each, and the groups of L lanes of all four wavefronts share the work, in the far part the
// boxes of the interaction lists and in the direct part the sources; the groups' sums are added at the end.  (With one
// target per lane and 64 per wavefront, leaves of about 20 points left two thirds of the lanes repeating the others'
// boxes; with L fixed at 8 a leaf of 22 points was two parts that staged every box twice, two lanes of five empty; and
// with a wavefront to itself a part is so much work that the last of 1.4 rounds of wavefronts left the chip half idle.)
// The list of boxes is made level by level with one candidate per lane.  Each step of a wavefront stages the
// coefficients of its groups' boxes (rows M, D and M / k) in LDS, read from memory one step ahead; the three Horner
// chains use each coefficient for both targets of a lane.  What bounds it is float64 VALU issue (143 of 237 us at
// 89,457 ragged points, order 20, depth 6) and the latency of a step at three wavefronts per SIMD.
// The kernel there: 337 -> 237 us.  Whole calls: 580 -> 283 us; 29,283 points, order 30, 347 -> 156 us; 8,192, order
// 12, 105 -> 63 us; 2000 x 128, order 30, 1.26 -> 0.99 ms.
constexpr int kTreeT = 2;  // targets per lane
constexpr int kTreeChunkShift = 5;  // log2 of the most targets per wavefront
constexpr int kTreeWaves = 4;       // wavefronts that share a part
constexpr int kTreeMinLanes = 8, kTreeMaxGroups = 64 / kTreeMinLanes;

constexpr int kListMax = 27 * (kMaxDepth - 1);     // boxes of all interaction lists of a leaf

// Box of a list entry: level in bits 20-23, column in 10-19, row in 0-9.
__device__ __forceinline__ int list_entry(int l, int sx, int sy) { return l << 20 | sx << 10 | sy; }

// a = a t + c in four three-address FMAs.  (The compiler's two-address form needs a copy of every c but for its last
// user, and one of every sum at the end of the loop: 21 instructions beside 24 FMAs.)
__device__ __forceinline__ void horner_step(double2& a, double2 t, double2 c) {
  double2 r;
  asm("v_fma_f64 %0, -%1, %2, %3" : "=v"(r.x) : "v"(a.y), "v"(t.y), "v"(c.x));
  asm("v_fma_f64 %0, %1, %2, %3" : "=v"(r.y) : "v"(a.y), "v"(t.x), "v"(c.y));
  asm("v_fma_f64 %0, %1, %2, %3" : "=v"(a.y) : "v"(a.x), "v"(t.y), "v"(r.y));
  asm("v_fma_f64 %0, %1, %2, %3" : "=v"(a.x) : "v"(a.x), "v"(t.x), "v"(r.x));
}

// kAhead: entries of a step's coefficients per lane.
template <int kAhead>
__global__ __launch_bounds__(64 * kTreeWaves) void k_tc_eval(const double4* __restrict__ srec, const int32_t* __restrict__ svid,
                                                int P, const int32_t* __restrict__ perm,
                                                const int32_t* __restrict__ starts,
                                                const int32_t* __restrict__ wstart, const Geom* __restrict__ geom,
                                                int depth, int p, const double2* __restrict__ mom,
                                                const int32_t* __restrict__ bcount, double scale,
                                                int max_groups, double* __restrict__ out) {
  extern __shared__ double2 cfs[];  // [kTreeWaves][max_groups][3 (p + 1)] coefficients of the step's boxes
  __shared__ int32_t list[kListMax + 1];
  __shared__ unsigned first[kListMax + 1];  // of the boxes' moments
  __shared__ double4 srcs[kTreeWaves][64];
  __shared__ int32_t svs[kTreeWaves][64];
  __shared__ double2 ltab[kLogTab];
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
  double2* cf = cfs + (size_t)wave * max_groups * 3 * (p + 1);
  double4* src = srcs[wave];
  int32_t* sv = svs[wave];
  const int n = 1 << depth;
  const int nleaf = n * n;
  const int item = blockIdx.x;
  if (item >= wstart[nleaf]) return;
  const int leaf = leaf_of_item(wstart, nleaf, item);
  const int s0 = starts[leaf], count = starts[leaf + 1] - s0;
  const int part = item - wstart[leaf], parts = wstart[leaf + 1] - wstart[leaf];
  const int base = s0 + (int)((int64_t)count * part / parts), s1 = s0 + (int)((int64_t)count * (part + 1) / parts);
  const int lanes = max((s1 - base + kTreeT - 1) / kTreeT, kTreeMinLanes), groups = min(64 / lanes, max_groups);
  const int grp = lane / lanes, tl = lane - grp * lanes;  // grp = groups: no work
  const int mine = wave * groups, step = kTreeWaves * groups;  // this wavefront's first group of all
  if (wave == 0) ltab[lane] = log_tab_entry(lane);
  double zx[kTreeT], zy[kTreeT], ux[kTreeT], uy[kTreeT];
  int ti[kTreeT], vi[kTreeT];
#pragma unroll
  for (int k = 0; k < kTreeT; ++k) {
    const int slot = base + tl + lanes * k;
    const int sl = slot < s1 ? slot : base;  // an empty slot repeats the first target
    ti[k] = perm[sl];
    const double4 z = srec[sl];
    zx[k] = z.x;
    zy[k] = z.y;
    vi[k] = svid[sl];
    ux[k] = uy[k] = 0.0;
  }
  const int ix = leaf / n, iy = leaf % n;
  const Geom g = *geom;
  // the non-empty boxes of the interaction lists, levels 2 .. depth: lane c examines candidate c of a level
  int nbox = 0;
  for (int l = 2; l <= depth; ++l) {
    const int nl = 1 << l, bx = ix >> (depth - l), by = iy >> (depth - l);
    const int sx = 2 * (bx >> 1) + lane / 6 - 2, sy = 2 * (by >> 1) + lane % 6 - 2;
    bool ok = lane < 36 && sx >= 0 && sx < nl && sy >= 0 && sy < nl && (abs(sx - bx) > 1 || abs(sy - by) > 1);
    if (ok) ok = bcount[level_box_base(l) + (size_t)sx * nl + sy] != 0;
    const unsigned long long m = __ballot(ok);
    if (ok && wave == 0) {
      const int at = nbox + __popcll(m & ((1ull << lane) - 1ull));
      list[at] = list_entry(l, sx, sy);
      first[at] = (unsigned)(level_box_base(l) + (size_t)sx * nl + sy) * 4 * (unsigned)(p + 1);
    }
    nbox += __popcll(m);
  }
  __syncthreads();
  const int np = p + 1, row3 = 3 * np;
  // Entry e of a step's coefficients: box e / (3 np), then rows M, D, M / k (rows 0, 2 and 3 of the moments).  A lane's
  // entries have the same place in every step: box << 16 | offset in the box.
  int place[kAhead];
#pragma unroll
  for (int u = 0; u < kAhead; ++u) {
    const int e = lane + 64 * u, b = e / row3, r = e - b * row3;
    place[u] = b < groups ? b << 16 | (r + (r >= np ? np : 0)) : 0;
  }
  double2 ahead[kAhead];  // the next step's entries, read while this step's are used
  const auto entry = [&](int b0, int pl) __attribute__((always_inline)) {
    return mom[first[min(b0 + (pl >> 16), nbox - 1)] + (pl & 0xffff)];
  };
  if (nbox > 0) {
#pragma unroll
    for (int u = 0; u < kAhead; ++u) ahead[u] = entry(mine, place[u]);
  }
  for (int b0 = mine; b0 < nbox; b0 += step) {
    wave_sync();  // the previous step is done with cf
    const int cnt = min(groups, nbox - b0) * row3;
#pragma unroll
    for (int u = 0; u < kAhead; ++u)
      if (lane + 64 * u < cnt) cf[lane + 64 * u] = ahead[u];
    wave_sync();
#pragma unroll
    for (int u = 0; u < kAhead; ++u) ahead[u] = entry(b0 + step, place[u]);  // past the end: the last box
    if (grp < groups && b0 + grp < nbox) {
      const int en = list[b0 + grp];
      const double2 c = box_center(g, 1 << (en >> 20), (en >> 10) & 1023, en & 1023);
      const double2* cb = cf + grp * row3;
      // Three series in t = 1 / w, highest order first:
      //   S = sum_{k>=1} M_k[F] / k t^k,  D = sum_k D_k t^(k+1),  E = sum_k M_k[F] t^k;
      // the box contributes S/2 + M_0/2 - M_0 ln|w| + conj(D) + (w / conj w) conj(E) / 2.
      double2 wv[kTreeT], t[kTreeT], aS[kTreeT], aD[kTreeT], aE[kTreeT];
      double w2[kTreeT], rw[kTreeT];
#pragma unroll
      for (int k = 0; k < kTreeT; ++k) {
        wv[k] = make_double2(zx[k] - c.x, zy[k] - c.y);
        w2[k] = wv[k].x * wv[k].x + wv[k].y * wv[k].y;
        rw[k] = recip(w2[k]);
        t[k] = make_double2(wv[k].x * rw[k], -wv[k].y * rw[k]);
        aS[k] = aD[k] = aE[k] = make_double2(0.0, 0.0);
      }
#pragma unroll 2
      for (int q = p; q >= 1; --q) {
        const double2 cE = cb[q], cD = cb[np + q], cS = cb[2 * np + q];
#pragma unroll
        for (int k = 0; k < kTreeT; ++k) {
          horner_step(aS[k], t[k], cS);
          horner_step(aD[k], t[k], cD);
          horner_step(aE[k], t[k], cE);
        }
      }
      const double2 M0 = cb[0], D0 = cb[np];
#pragma unroll
      for (int k = 0; k < kTreeT; ++k) {
        const double2 e = cfma(aE[k], t[k], M0);
        const double2 d = cmul(cfma(aD[k], t[k], D0), t[k]);
        const double2 sS = cmul(aS[k], t[k]);
        const double lnw = 0.5 * log_reduced(w2[k], ltab);
        const double2 rot = make_double2((wv[k].x * wv[k].x - wv[k].y * wv[k].y) * rw[k],
                                         2.0 * wv[k].x * wv[k].y * rw[k]);  // w / conj w
        const double2 pe = cmul(rot, make_double2(e.x, -e.y));
        ux[k] += 0.5 * sS.x + 0.5 * M0.x - M0.x * lnw + d.x + 0.5 * pe.x;
        uy[k] += 0.5 * sS.y + 0.5 * M0.y - M0.y * lnw - d.y + 0.5 * pe.y;
      }
    }
  }
  // 3 x 3 leaves directly, own vesicle skipped: the three leaves of a column are one run of the leaf order
  for (int jx = max(ix - 1, 0); jx <= min(ix + 1, n - 1); ++jx) {
    const int e0 = starts[jx * n + max(iy - 1, 0)], e1 = starts[jx * n + min(iy + 1, n - 1) + 1];
    for (int c0 = e0; c0 < e1; c0 += 64) {
      const int cnt = min(64, e1 - c0);
      wave_sync();  // the previous chunk is done
      if (lane < cnt) {
        src[lane] = srec[c0 + lane];
        sv[lane] = svid[c0 + lane];
      }
      wave_sync();
      for (int q = grp < groups ? mine + grp : cnt; q < cnt; q += step) {
        const double4 s = src[q];
        const int cv = sv[q];
#pragma unroll
        for (int k = 0; k < kTreeT; ++k)
          if (cv != vi[k]) direct_term(zx[k], zy[k], s.x, s.y, s.z, s.w, ltab, ux[k], uy[k]);
      }
    }
  }
  wave_sync();  // the records are done: their place holds the groups' sums, added in order
  src[lane] = make_double4(ux[0], uy[0], ux[1], uy[1]);
  __syncthreads();
  if (wave > 0 || grp > 0) return;
  for (int q = 1; q < step; ++q) {
    const double4 u = srcs[q / groups][(q % groups) * lanes + tl];
    ux[0] += u.x;
    uy[0] += u.y;
    ux[1] += u.z;
    uy[1] += u.w;
  }
#pragma unroll
  for (int k = 0; k < kTreeT; ++k)
    if (base + tl + lanes * k < s1) {
      out[ti[k]] += ux[k] * scale;  // to the own-vesicle terms
      out[P + ti[k]] += uy[k] * scale;
    }
}

// Near-field masking of Algorithm 4 on the fast multipole result: vesicle v (not the target's own) is near
// target i when min_j |x_i - x_j| <= h_v (the rule of the direct masked sum, decided here in FP64 on
// squared distances).  With every h_v at most the leaf width, all such points lie in the 3 x 3 leaves around
// the target's leaf.  One wavefront per (leaf, chunk of targets: the evaluation's work list), four to a workgroup,
// stages those leaves' records in LDS, up to kNearStage at a time with every lane's loads issued together; the 64 /
// chunk lanes t, t + chunk, ... scan interleaved points for target t, each keeping the distinct near vesicles it meets
// (at most kNearMax, else bit 0 of *flag), and lane t merges the sets and sorts them ascending.  One atomic per
// workgroup reserves the pair slots (they all go to one address, about 20 ns each).  The lanes of a target then share
// the points of its near vesicles and subtract their exact direct sum at x_i from out[i]: the FMM had included v
// through the direct part or the expansions, and the difference leaves the masked far field with the FMM's
// truncation error.  The lane partials are combined by a butterfly, so the result is deterministic.
// 2000 x 32: 56 -> 32 us (before: one atomic per wavefront; the whole wavefront on one target after the other, a
// memory latency each; points gathered through the permutation).  Five workgroups per compute unit: with the 124
// registers that the compiler takes unasked it is four, and 36 us.
constexpr int kNearMax = 16;
constexpr int kNearStage = 4 * 64;  // points of the 3 x 3 leaves staged at once (four per lane)

__device__ __forceinline__ void near_insert(int (&nv)[kNearMax], int& nn, bool& over, int v) {
  bool seen = false;
#pragma unroll
  for (int k = 0; k < kNearMax; ++k) seen |= k < nn && nv[k] == v;
  if (seen) return;
  if (nn == kNearMax) {
    over = true;
    return;
  }
#pragma unroll
  for (int k = 0; k < kNearMax; ++k)
    if (k == nn) nv[k] = v;
  ++nn;
}

constexpr int kNearWaves = 4;

__global__ __launch_bounds__(64 * kNearWaves, 5) void k_fmm_near(const double* __restrict__ X, const double* __restrict__ f,
                                                const double* __restrict__ w, int P, int M,
                                                const int32_t* __restrict__ off,
                                                const double4* __restrict__ srec, const int32_t* __restrict__ svid,
                                                const int32_t* __restrict__ perm, const int32_t* __restrict__ starts,
                                                const int32_t* __restrict__ wstart, int depth,
                                                const double* __restrict__ h2, double scale, double* __restrict__ out,
                                                int32_t* __restrict__ pairs, int capacity, int32_t* __restrict__ count,
                                                int32_t* __restrict__ flag) {
  constexpr int kChunk = 1 << kFmmChunkShift;
  constexpr int kGroups = 64 / kChunk;  // lanes per target: group g scans every kGroups-th source from g on
  static_assert(kGroups >= 2 && kGroups * kChunk == 64, "a power-of-two chunk of at most 32 targets");
  // a wavefront's staged records, then its groups' sets
  struct Stage {
    double x[kNearStage], y[kNearStage], h2[kNearStage];
    int32_t v[kNearStage];
  };
  struct Sets {
    int32_t list[kGroups - 1][kChunk][kNearMax + 1], count[kGroups - 1][kChunk];
  };
  union Shared {
    Stage st;
    Sets se;
    __device__ Shared() {}
  };
  __shared__ Shared shared[kNearWaves];
  __shared__ double2 ltab[kLogTab];
  __shared__ int32_t found[kNearWaves], first;
  const int n = 1 << depth;
  const int nleaf = n * n;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
  const int item = blockIdx.x * kNearWaves + wave;
  if (threadIdx.x < kLogTab) ltab[threadIdx.x] = log_tab_entry(threadIdx.x);  // read after the barriers below
  const bool some = item < wstart[nleaf];  // a wavefront without an item takes a chunk beyond its leaf's last
  const int leaf = some ? leaf_of_item(wstart, nleaf, item) : 0;
  Stage& st = shared[wave].st;
  Sets& se = shared[wave].se;
  const int t = lane & (kChunk - 1), grp = lane / kChunk;
  const int s0 = starts[leaf], s1 = starts[leaf + 1];
  const int slot = s0 + (item - wstart[leaf]) * kChunk + t;
  const bool active = some && slot < s1;
  const int sl = active ? slot : min(s0, P - 1);
  const int i = perm[sl];
  const double zx = srec[sl].x, zy = srec[sl].y;
  const int vi = clamp_i(svid[sl], 0, M - 1);
  const int ix = leaf / n, iy = leaf % n;
  int nv[kNearMax];
  int nn = 0;
  bool over = false;
  // the source runs of columns ix - 1 .. ix + 1 (empty outside the grid), as one list of nsrc slots
  int run0[3], cum[4];
  cum[0] = 0;
#pragma unroll
  for (int a = 0; a < 3; ++a) {
    const int jx = ix + a - 1;
    const bool in = jx >= 0 && jx < n;
    run0[a] = in ? starts[jx * n + max(iy - 1, 0)] : 0;
    cum[a + 1] = cum[a] + (in ? starts[jx * n + min(iy + 1, n - 1) + 1] - run0[a] : 0);
  }
  const int nsrc = some ? cum[3] : 0;
  for (int b0 = 0; b0 < nsrc; b0 += kNearStage) {
    const int cnt = min(kNearStage, nsrc - b0);
    double2 pos[kNearStage / 64];
    int vv[kNearStage / 64];
#pragma unroll
    for (int u = 0; u < kNearStage / 64; ++u) {
      const int e = min(b0 + lane + 64 * u, nsrc - 1);
      const int at = e < cum[1] ? run0[0] + e : e < cum[2] ? run0[1] + e - cum[1] : run0[2] + e - cum[2];
      pos[u] = make_double2(srec[at].x, srec[at].y);
      vv[u] = clamp_i(svid[at], 0, M - 1);  // ids index the per-vesicle arrays: never trusted
    }
    wave_sync();  // the previous stage is done
#pragma unroll
    for (int u = 0; u < kNearStage / 64; ++u) {
      const int k = lane + 64 * u;
      st.x[k] = pos[u].x;
      st.y[k] = pos[u].y;
      st.v[k] = vv[u];
      st.h2[k] = h2[vv[u]];
    }
    wave_sync();
    if (active) {
#pragma unroll 4
      for (int q = grp; q < cnt; q += kGroups) {
        const double rx = zx - st.x[q], ry = zy - st.y[q];
        const int vq = st.v[q];
        if (!(rx * rx + ry * ry > st.h2[q]) && vq != vi) near_insert(nv, nn, over, vq);
      }
    }
  }
  wave_sync();  // the staged records are done: their place now holds the sets
  // merge the other groups' sets into group 0's
  if (grp > 0) {
#pragma unroll
    for (int k = 0; k < kNearMax; ++k)
      if (k < nn) se.list[grp - 1][t][k] = nv[k];
    se.count[grp - 1][t] = nn;
    nn = 0;
  }
  wave_sync();
  if (grp == 0)
    for (int g2 = 0; g2 < kGroups - 1; ++g2) {
      const int m = se.count[g2][t];
      for (int k = 0; k < m; ++k) near_insert(nv, nn, over, se.list[g2][t][k]);
    }
  int most = 0;  // largest set of the wavefront
  while (__ballot(nn > most) != 0) ++most;
  // ascending vesicle order: the subtraction order, and so the result, does not depend on the scan
#pragma unroll
  for (int a = 1; a < kNearMax; ++a)
    if (a < most) {
#pragma unroll
      for (int b = kNearMax - 1; b >= a; --b)
        if (b < nn && nv[b - 1] > nv[b]) {
          const int tmp = nv[b - 1];
          nv[b - 1] = nv[b];
          nv[b] = tmp;
        }
    }
  if (__ballot(over) != 0 && lane == 0) atomicOr(flag, 1);
  int incl = nn;  // inclusive prefix of the pair counts over the wavefront (zero outside group 0)
  for (int o = 1; o < kChunk; o <<= 1) {
    const int y = __shfl_up(incl, o);
    if (lane >= o) incl += y;
  }
  if (lane == kChunk - 1) found[wave] = incl;
  __syncthreads();
  int total = 0, before = 0;
#pragma unroll
  for (int q = 0; q < kNearWaves; ++q) {
    if (q < wave) before += found[q];
    total += found[q];
  }
  if (total == 0) return;
  if (threadIdx.x == 0) first = atomicAdd(count, total);
  __syncthreads();
  if (grp == 0) {
    const int b0 = first + before + incl - nn;
#pragma unroll
    for (int k = 0; k < kNearMax; ++k)
      if (k < nn) {
        if (b0 + k < capacity) {
          pairs[2 * (b0 + k)] = i;
          pairs[2 * (b0 + k) + 1] = nv[k];
        }
        se.list[0][t][k] = nv[k];
      }
    se.count[0][t] = nn;
  }
  wave_sync();
  const int m = se.count[0][t];
  double ux = 0.0, uy = 0.0;
  for (int k = 0; k < m; ++k) {
    const int v = se.list[0][t][k];
    const int v0 = clamp_i(off[v], 0, P), v1 = max(v0, clamp_i(off[v + 1], 0, P));
#pragma unroll 4
    for (int j = v0 + grp; j < v1; j += kGroups)
      direct_term(zx, zy, X[j], X[P + j], w[j] * f[j], w[j] * f[P + j], ltab, ux, uy);
  }
#pragma unroll
  for (int o = kChunk; o < 64; o <<= 1) {
    ux += __shfl_xor(ux, o);
    uy += __shfl_xor(uy, o);
  }
  if (grp == 0 && nn > 0) {
    out[i] -= ux * scale;
    out[P + i] -= uy * scale;
  }
}

// The list's status: a negative count when the masking could not be completed (see k_fmm_near and k_tc_leaf).
__global__ __launch_bounds__(64) void k_fmm_near_status(const int32_t* __restrict__ flag, int32_t* __restrict__ count) {
  if (threadIdx.x != 0) return;
  const int32_t fl = *flag;
  if (fl & 2) *count = -2;
  else if (fl & 1) *count = -1;
}

}  // namespace

// Workspace layout shared by the size queries and the launchers; the fast multipole method adds the
// local expansions (3 rows per box) and the evaluation's log table.
struct TreeLayout {
  size_t geom, part, leafid, vid, perm, srec, svid, counts, starts, wstart, bcount, mom, loc, ltab, h2, flag,
      total;
};

static size_t align_up(size_t x) { return (x + 255) / 256 * 256; }

static TreeLayout tree_layout(int P, int depth, int p, bool fmm, int near_M = 0) {
  TreeLayout t;
  const size_t nleaf = (size_t)1 << (2 * depth);
  size_t boxes = 0;
  for (int l = 2; l <= depth; ++l) boxes += (size_t)1 << (2 * l);
  const size_t moms = boxes * 4 * (size_t)(p + 1);
  size_t o = 0;
  t.geom = o;       o += align_up(sizeof(double) * 4);
  t.part = o;       o += align_up(sizeof(double) * 4 * kBBoxBlocks);
  t.leafid = o;     o += align_up(sizeof(int32_t) * (size_t)P);
  t.vid = o;        o += align_up(sizeof(int32_t) * (size_t)P);
  t.perm = o;       o += align_up(sizeof(int32_t) * (size_t)P);
  t.srec = o;       o += align_up(sizeof(double4) * (size_t)P);
  t.svid = o;       o += align_up(sizeof(int32_t) * (size_t)P);
  t.counts = o;     o += align_up(sizeof(int32_t) * nleaf);
  t.starts = o;     o += align_up(sizeof(int32_t) * (nleaf + 1));
  t.wstart = o;     o += align_up(sizeof(int32_t) * (nleaf + 1));
  t.bcount = o;     o += align_up(sizeof(int32_t) * (boxes > 0 ? boxes : 1));
  t.mom = o;        o += align_up(sizeof(double2) * (moms + 256));  // 256 spare entries: whole-wave copies
  t.loc = o;
  t.ltab = o;
  if (fmm) {
    t.loc = o;      o += align_up(sizeof(double2) * (boxes * 3 * (size_t)(p + 1) + 192));  // 192 spare: as above
    t.ltab = o;     o += align_up(sizeof(double2) * (size_t)kHalfLogTab);
  }
  t.h2 = o;
  t.flag = o;
  if (near_M > 0) {  // near-field masking: h_v^2 of every vesicle and a status word
    t.h2 = o;       o += align_up(sizeof(double) * (size_t)near_M);
    t.flag = o;     o += align_up(sizeof(int32_t));
  }
  t.total = o;
  return t;
}

size_t treecode_workspace_bytes(int P, int depth, int p) { return tree_layout(P, depth, p, false).total; }
size_t fmm_workspace_bytes(int P, int depth, int p) { return tree_layout(P, depth, p, true).total; }
size_t fmm_near_workspace_bytes(int P, int M, int depth, int p) { return tree_layout(P, depth, p, true, M).total; }

namespace {

struct TreeRun {
  Geom* geom;
  double* part;
  int32_t *leafid, *vid, *perm, *counts, *starts, *wstart, *bcount;
  double4* srec;   // records and vesicle ids in leaf order
  int32_t* svid;
  double2 *mom, *loc, *ltab;
  double* h2;
  int32_t* flag;
  Levels lv;       // first box and first moment entry of every level
  size_t nbox;     // boxes of levels 2..depth
};

TreeRun tree_run(void* ws, const TreeLayout& t, int depth, int p) {
  char* base = static_cast<char*>(ws);
  TreeRun r;
  r.geom = reinterpret_cast<Geom*>(base + t.geom);
  r.part = reinterpret_cast<double*>(base + t.part);
  r.leafid = reinterpret_cast<int32_t*>(base + t.leafid);
  r.vid = reinterpret_cast<int32_t*>(base + t.vid);
  r.perm = reinterpret_cast<int32_t*>(base + t.perm);
  r.srec = reinterpret_cast<double4*>(base + t.srec);
  r.svid = reinterpret_cast<int32_t*>(base + t.svid);
  r.ltab = reinterpret_cast<double2*>(base + t.ltab);
  r.counts = reinterpret_cast<int32_t*>(base + t.counts);
  r.starts = reinterpret_cast<int32_t*>(base + t.starts);
  r.wstart = reinterpret_cast<int32_t*>(base + t.wstart);
  r.bcount = reinterpret_cast<int32_t*>(base + t.bcount);
  r.mom = reinterpret_cast<double2*>(base + t.mom);
  r.loc = reinterpret_cast<double2*>(base + t.loc);
  r.h2 = reinterpret_cast<double*>(base + t.h2);
  r.flag = reinterpret_cast<int32_t*>(base + t.flag);
  r.lv = {};
  size_t acc = 0;
  for (int l = 2; l <= depth; ++l) {  // boxes of level l start at box index sum_{m = 2}^{l-1} 4^m
    r.lv.box[l] = acc;
    r.lv.mom[l] = acc * 4 * (size_t)(p + 1);
    acc += (size_t)1 << (2 * l);
  }
  r.nbox = acc;
  return r;
}

// Tree over the points (root square, leaves, leaf order) and the moments of every box of levels
// 2..depth (leaves from the points, coarser levels by translation).
void launch_upward(const double* X, const double* f, const double* w, const int32_t* off, int M, int P, int p,
                   int depth, int cshift, bool fmm, int32_t* count, double scale, double* out, const TreeRun& r,
                   hipStream_t st) {
  const int nleaf = 1 << (2 * depth);
  const int pb = (P + kTB - 1) / kTB < 4096 ? (P + kTB - 1) / kTB : 4096;
  const int bb = (P + kTB - 1) / kTB < kBBoxBlocks ? (P + kTB - 1) / kTB : kBBoxBlocks;
  hipLaunchKernelGGL(k_tc_bbox_partial, dim3(bb), dim3(kTB), 0, st, X, P, r.part, fmm ? r.ltab : nullptr, r.counts,
                     nleaf, count, r.flag);
  hipLaunchKernelGGL(k_tc_leaf, dim3(pb + M), dim3(kTB), 0, st, X, P, r.part, bb, pb, depth, r.geom, r.leafid, r.counts,
                     r.svid /* places, until the sort */, off, r.vid, w, count ? r.h2 : nullptr, r.flag, out);
  hipLaunchKernelGGL(k_tc_scan, dim3(1), dim3(1024), 0, st, r.counts, nleaf, r.starts, r.wstart, cshift);
  hipLaunchKernelGGL(k_tc_scatter, dim3(pb), dim3(kTB), 0, st, r.leafid, P, r.starts, r.svid, r.perm);
  hipLaunchKernelGGL(k_tc_sort, dim3(nleaf), dim3(64), 0, st, X, f, w, P, r.vid, r.starts, r.perm, r.srec, r.svid);
  if (depth < 2) return;
  const bool up = depth > 2;
  const dim3 pg(nleaf / 4 + (M + 1) / 2), pbl(256);
  double2* pmom = up ? r.mom + r.lv.mom[depth - 1] : nullptr;
  int32_t* pcount = up ? r.bcount + r.lv.box[depth - 1] : nullptr;
  // The leaves and their parents, then the coarser levels, two to a launch: one box of the upper level has four below,
  // whose sixteen children are one pass of a workgroup (3 us; with three levels to a launch, four passes for the lowest:
  // 26 instead of 18 us at depth 6).
#define VESNET_UP(K)                                                                                                \
  case K:                                                                                                           \
    hipLaunchKernelGGL(k_tc_p2m<K>, pg, pbl, 0, st, r.srec, r.starts, r.geom, depth, p, r.mom + r.lv.mom[depth],    \
                       r.bcount + r.lv.box[depth], pmom, pcount, !fmm, X, f, w, P, off, M, r.leafid, scale, out);   \
    for (int l = depth - 2, to; l >= 2; l = to - 1) {                                                               \
      to = l > 2 ? l - 1 : 2;                                                                                       \
      hipLaunchKernelGGL(k_tc_m2m<K>, dim3(1 << (2 * to)), dim3(l > to ? 64 * up_waves(K) : 256), 0, st, r.geom, l, to, \
                         p, r.mom, r.bcount, !fmm);                                                                 \
    }                                                                                                               \
    break;
  switch ((p + 8) / 8) {  // orders per lane: ceil((p + 1) / 8)
    VESNET_UP(1) VESNET_UP(2) VESNET_UP(3) VESNET_UP(4) VESNET_UP(5) VESNET_UP(6) VESNET_UP(7)
  }
#undef VESNET_UP
}

// Work items of an evaluation: a bound on sum over leaves of ceil(count / 2^shift).
int eval_items(int P, int depth, int shift) { return (1 << (2 * depth)) + ((P + (1 << shift) - 1) >> shift); }

}  // namespace

// Everything is built on the device; the launches need no host copy and no synchronisation.
hipError_t launch_treecode(const double* X, const double* f, const double* w, const int32_t* off, int M, int P,
                           double scale, int p, int depth, double* out, void* ws, void* stream) {
  if (P == 0) return hipSuccess;
  if (depth < 0 || depth > kMaxDepth || p < 1 || p > kMaxOrder) return hipErrorInvalidValue;
  hipStream_t st = reinterpret_cast<hipStream_t>(stream);
  const TreeRun r = tree_run(ws, tree_layout(P, depth, p, false), depth, p);
  launch_upward(X, f, w, off, M, P, p, depth, kTreeChunkShift, false, nullptr, scale, out, r, st);
  // groups whose boxes fit 48 KB: all eight up to order 31, five at 48
  const size_t per = sizeof(double2) * (size_t)kTreeWaves * 3 * (p + 1);
  const int max_groups = (size_t)kTreeMaxGroups * per <= 49152 ? kTreeMaxGroups : (int)(49152 / per);
  const dim3 grid((unsigned)eval_items(P, depth, kTreeChunkShift)), block(64 * kTreeWaves);
  if (max_groups * 3 * (p + 1) <= 8 * 64)
    hipLaunchKernelGGL(k_tc_eval<8>, grid, block, per * max_groups, st, r.srec, r.svid, P, r.perm, r.starts, r.wstart,
                       r.geom, depth, p, r.mom, r.bcount, scale, max_groups, out);
  else
    hipLaunchKernelGGL(k_tc_eval<12>, grid, block, per * max_groups, st, r.srec, r.svid, P, r.perm, r.starts, r.wstart,
                       r.geom, depth, p, r.mom, r.bcount, scale, max_groups, out);
  return hipGetLastError();
}

static hipError_t run_fmm(const double* X, const double* f, const double* w, const int32_t* off, int M, int P,
                          double scale, int p, int depth, double* out, void* ws, hipStream_t st, bool near,
                          int32_t* pairs, int capacity, int32_t* count) {
  const TreeRun r = tree_run(ws, tree_layout(P, depth, p, true, near ? M : 0), depth, p);
  launch_upward(X, f, w, off, M, P, p, depth, kFmmChunkShift, true, near ? count : nullptr, scale, out, r, st);
  if (depth >= 2) {
    const dim3 g((unsigned)r.nbox), bl(64);
    const size_t lds = m2l_lds_bytes(p);
    switch (m2l_rtiles(p)) {
      case 1: hipLaunchKernelGGL(k_fmm_m2l<1>, g, bl, lds, st, r.geom, depth, p, r.mom, r.bcount, r.loc); break;
      case 2: hipLaunchKernelGGL(k_fmm_m2l<2>, g, bl, lds, st, r.geom, depth, p, r.mom, r.bcount, r.loc); break;
      case 3: hipLaunchKernelGGL(k_fmm_m2l<3>, g, bl, lds, st, r.geom, depth, p, r.mom, r.bcount, r.loc); break;
      default: hipLaunchKernelGGL(k_fmm_m2l<4>, g, bl, lds, st, r.geom, depth, p, r.mom, r.bcount, r.loc); break;
    }
    if (depth >= 3) {
      const int nleaf = 1 << (2 * depth);
#define VESNET_L2L(K)                                                                                              \
  case K:                                                                                                          \
    hipLaunchKernelGGL(k_fmm_l2l<K>, dim3(nleaf / kShiftWaves), dim3(64 * kShiftWaves), 0, st, r.geom, depth, p,   \
                       r.bcount, r.loc);                                                                           \
    break;
      switch ((p + 8) / 8) {  // ceil((p + 1) / 8)
        VESNET_L2L(1) VESNET_L2L(2) VESNET_L2L(3) VESNET_L2L(4) VESNET_L2L(5) VESNET_L2L(6) VESNET_L2L(7)
      }
#undef VESNET_L2L
    }
  }
  const int items = eval_items(P, depth, kFmmChunkShift);
  hipLaunchKernelGGL(k_fmm_eval, dim3((items + kFmmWaves - 1) / kFmmWaves), dim3(64 * kFmmWaves), 0, st, r.srec, r.svid,
                     P, r.perm, r.starts, r.wstart, r.geom, depth, p, r.loc, r.ltab, scale, out);
  if (near) {
    hipLaunchKernelGGL(k_fmm_near, dim3((items + kNearWaves - 1) / kNearWaves), dim3(64 * kNearWaves), 0, st, X, f, w, P, M, off, r.srec, r.svid, r.perm, r.starts,
                       r.wstart, depth, r.h2, scale, out, pairs, capacity, count, r.flag);
    hipLaunchKernelGGL(k_fmm_near_status, dim3(1), dim3(64), 0, st, r.flag, count);
  }
  return hipGetLastError();
}

hipError_t launch_fmm(const double* X, const double* f, const double* w, const int32_t* off, int M, int P,
                      double scale, int p, int depth, double* out, void* ws, void* stream) {
  if (P == 0) return hipSuccess;
  if (depth < 0 || depth > kMaxDepth || p < 1 || p > kMaxOrder) return hipErrorInvalidValue;
  return run_fmm(X, f, w, off, M, P, scale, p, depth, out, ws, reinterpret_cast<hipStream_t>(stream), false, nullptr,
                 0, nullptr);
}

hipError_t launch_zero_count(int32_t* count, void* stream) {
  hipLaunchKernelGGL(k_tc_zero, dim3(1), dim3(64), 0, reinterpret_cast<hipStream_t>(stream), count);
  return hipGetLastError();
}

hipError_t launch_fmm_nearmasked(const double* X, const double* f, const double* w, const int32_t* off, int M, int P,
                                 double scale, int p, int depth, double* out, int32_t* pairs, int capacity,
                                 int32_t* count, void* ws, void* stream) {
  if (P == 0) return hipSuccess;
  if (depth < 0 || depth > kMaxDepth || p < 1 || p > kMaxOrder) return hipErrorInvalidValue;
  return run_fmm(X, f, w, off, M, P, scale, p, depth, out, ws, reinterpret_cast<hipStream_t>(stream), true, pairs,
                 capacity, count);
}

}  // namespace vesnet

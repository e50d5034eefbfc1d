// Symmetric far-field kernels for gfx950: each unordered cross-vesicle pair is evaluated once.
//
// The Stokeslet of eq. (Stokeslet), read as -ln|r| I + r r^T/|r|^2, is even in r, and the
// trapezoid sum of eq. (single_layer) (Section 2.2.1) taken at the discretisation points
// themselves uses every point as target and as source.  One evaluation of r, |r|^2, its
// logarithm and its reciprocal therefore serves both ordered pairs (i <- j and j <- i), which
// halves the transcendental instructions of the direct gather (26 issue slots per unordered pair,
// 13 per ordered pair, against 19.6).
// This file holds, on one schedule: the float32-compensated forward (k_sym_main) and its batched
// persistent form (k_symb_*), the float64 forward (k_sym64_main), and the adjoints of one point
// array in float32-compensated (k_sym_bwd) and float64 (k_sym64_bwd) form.  The description below is
// the float32-compensated forward's; the other kernels state where they differ.
//
// Work decomposition
//  * Points are cut into "cycles" of at most 16 consecutive points of one vesicle (a vesicle of
//    N points gives ceil(N/16) cycles); CB = 16 T consecutive cycles form a block.
//  * A unit is an unordered pair of blocks {bx, by}, by = bx + d (mod nb), d = 0 .. nb/2 (the
//    circulant schedule visits every unordered pair of blocks once; for even nb the pairs at
//    d = nb/2 are taken by bx < nb/2 only).  One workgroup of 256 threads (4 wavefronts, 16 rows
//    of 16 lanes) evaluates a unit: row r holds target cycles r, r + 16, ... of block bx (T of
//    them, one point per lane), and the source cycles of block by stream through LDS in chunks
//    of 8 cycles.  With T = 3 (the float32-compensated default: 768-point blocks, 112 VGPRs, 32 KB of
//    LDS) four units share a compute unit; with T = 2 (512-point blocks, 94 VGPRs, 27 KB) five.
//  * Each row is a ring: at step s lane p pairs its T targets with source (p + s) mod 16 of the
//    current source cycle, read from LDS (each cycle is stored twice so that the address is the
//    lane's base plus an immediate offset).  The source's column sum travels with it around the
//    ring, by a DPP row rotation folded into the add that closes each step.  After 16 steps two
//    lane swaps (v_permlane32_swap, v_permlane16_swap) add the four rows of a wavefront, the
//    column sums go to LDS, and after each chunk the workgroup adds its 4 wavefronts in a fixed
//    order.
//  * Own vesicle and the diagonal unit (d = 0): a (target cycle, source vesicle) pair is active
//    when the vesicles differ and, for d = 0, when the target's vesicle index is the smaller one,
//    so every unordered cross-vesicle pair is evaluated once.  Inactive targets sit at a far
//    point with zero force: their column contributions are exact zeros and their row partials
//    are dropped by a select.  Slots of a cycle past its count hold a copy of the cycle's first
//    point with zero force (exact zeros in the rows; their column sums are never read).
//
// Compensation (float32 pairs, float64 corrections)
//  * For a target of vesicle A and a source vesicle B the pair loop runs on the rescaled
//    difference r' = 2^-k (x_i - y_j) = 2^-k (xi_i + c_A - c_B) - 2^-k xi_j, with xi the float32
//    local coordinates about each vesicle's point mean c (c_A - c_B rounded once from float64) and
//    k = floor(e/2) for |c_A - c_B|^2 + R_A^2 + R_B^2 = m 2^e (R the largest |xi| of a vesicle):
//    |r'| is of order one for distant vesicles and bounded for overlapping hulls.  Scaling by a
//    power of two is exact, so ln|r|^2 = ln 2 (log2|r'|^2 + 2k) exactly, and the rr-term is
//    unchanged.  (Plain subtractions on unscaled coordinates with the scale applied to |r|^2 give
//    the same bits but one more instruction per pair, and measured 4% slower.)
//  * Row (target, segment of B in the block): float32 partial of -1/2 ln2 log2|r'|^2 F_j + rr-term,
//    then in float64  - k ln2 F_seg, F_seg the float64 net force of the segment (the sum of its
//    cycles' float64 net forces).
//  * Column (source j of B, from the targets of one wavefront): float32 partial of the same terms
//    with the targets' forces; the log correction - ln2 sum_cycles k F_cycle (float64) is the same
//    for every source of B and is formed once per (wavefront, B).
//    A distant force-free vesicle's nearly constant log therefore never enters a float32 sum.
//
// Accumulation across workgroups is deterministic: every row and column partial is added in
// float64, rounded to a 64-bit fixed-point integer at 2^-S (S from a bound on every partial sum,
// 520 sum_j |F_j|_1 < 2^(62 - S)) and added with 64-bit integer atomics, whose result does not
// depend on their order.  A last kernel converts the integers back and scales by 1/(4 pi mu).
#include <hip/hip_runtime.h>
#include <math.h>
#include <stdint.h>

#include <algorithm>
#include <atomic>
#include <type_traits>

#include "vesnet_internal.h"

namespace vesnet {

namespace {

constexpr int kRing = 16;                          // sources per ring cycle (one DPP row)
constexpr int kXcds = 8;                           // XCDs of the MI355X (workgroups are dealt to them in turn)
constexpr int kSymThreads = 256;                   // threads per unit (4 wavefronts, one per SIMD)
constexpr int kSymWaves = kSymThreads / 64;
constexpr int kRows = kSymThreads / kRing;         // rows of 16 lanes per unit
constexpr int kChunk = 8;                          // source cycles per LDS chunk
static_assert(kChunk * 2 * kRing <= kSymThreads, "one thread per staged record and per column sum of a chunk");
constexpr double kLn2d = 0.69314718055994530942;
constexpr double kPi = 3.14159265358979323846;
constexpr float kHalfLn2f = -0.34657359027997265471f;  // -(1/2) ln 2: log2|r|^2 -> -ln|r|
constexpr float kFar = 1152921504606846976.0f;         // 2^60: position of an inactive target
constexpr int kMaxShift = 60;                          // |k| bound of the power-of-two rescaling

__device__ __forceinline__ float bitsf(unsigned x) { return __builtin_bit_cast(float, x); }
__device__ __forceinline__ unsigned bitsu(float x) { return __builtin_bit_cast(unsigned, x); }

// x from the lane one position up in the same row of 16 lanes (lane p reads lane (p + 1) mod 16).
__device__ __forceinline__ float ring_next(float x) {
  return bitsf((unsigned)__builtin_amdgcn_update_dpp(0, (int)bitsu(x), 0x12F, 0xF, 0xF, true));
}

__device__ __forceinline__ double wave_sum_d(double x) {
#pragma unroll
  for (int m = 32; m >= 1; m >>= 1) x += __shfl_xor(x, m, 64);
  return x;
}

// Fixed-point exponent of partial sums.  Every term of every one is at most (|ln q|/2 + 1) |F|_1 <= 520 |F|_1 in magnitude
// (log2|r'|^2 within the float32 range, |k| <= 60), so with 520 sum |F|_1 < 2^(62 - S) the fixed-point integers stay below
// 2^62.
__device__ __forceinline__ int sym_exponent(double fsum) {
  const double bound = 520.0 * fsum;
  if (!(bound > 0.0 && isfinite(bound))) return 0;
  int e;
  frexp(bound, &e);  // bound < 2^e
  return 62 - e;
}

// The same of the float64 form, also where 520 fsum overflows.
__device__ __forceinline__ int sym64_exponent(double fsum) {
  if (!(fsum > 0.0 && isfinite(fsum))) return 0;
  int e0, e;
  const double m = frexp(fsum, &e0);
  frexp(520.0 * m, &e);
  return 62 - e0 - e;
}

// A vesicle's share of that bound in the float64 form, a = sum |F|_1 over its points [r.x, r.y): none where a force is
// not finite, since every output that such a force enters is marked for it, and the vesicle's own keep their values.
// (An infinite share is the overflow of finite forces: then every output is NaN.)
__device__ __forceinline__ double bound_share(double a, int2 r, const double4* __restrict__ rec) {
  if (!isfinite(a))
    for (int j = r.x; j < r.y; ++j)
      if (!isfinite(rec[j].z) || !isfinite(rec[j].w)) return 0.0;
  return a;
}

// Plan: the cycle table of every vesicle in point order, the number of blocks and the
// fixed-point exponent.  One workgroup of 1024 threads; everything in a fixed order.
__global__ __launch_bounds__(1024) void k_sym_plan(const int2* __restrict__ vrange, const double2* __restrict__ vaux,
                                                   int M, int cb, int ncyc_max, int4* __restrict__ cyc,
                                                   int32_t* __restrict__ meta) {
  __shared__ int32_t s_wsum[16];
  __shared__ double s_dsum[16];
  const int t = threadIdx.x, lane = t & 63, wv = t >> 6;
  int run = 0;
  double fa = 0.0;
  for (int base = 0; base < M; base += 1024) {
    const int v = base + t;
    const int2 r = v < M ? vrange[v] : make_int2(0, 0);
    const int n = max(0, r.y - r.x);
    const int cnt = (n + kRing - 1) / kRing;
    if (v < M) fa += vaux[v].x;
    int x = cnt;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
      const int y = __shfl_up(x, o, 64);
      if (lane >= o) x += y;
    }
    if (lane == 63) s_wsum[wv] = x;
    __syncthreads();
    int pre = 0, tot = 0;
    for (int k = 0; k < 16; ++k) {
      const int s = s_wsum[k];
      pre += k < wv ? s : 0;
      tot += s;
    }
    const int first = run + pre + x - cnt;
    for (int c = 0; c < cnt; ++c) {
      const int e = first + c;
      if (e < ncyc_max) cyc[e] = make_int4(r.x + kRing * c, min(kRing, n - kRing * c), v, 0);
    }
    run += tot;
    __syncthreads();
  }
  fa = wave_sum_d(fa);
  if (lane == 0) s_dsum[wv] = fa;
  __syncthreads();
  if (t == 0) {
    double tot = 0.0;
    for (int k = 0; k < 16; ++k) tot += s_dsum[k];
    const int ncyc = min(run, ncyc_max);
    meta[0] = ncyc;
    meta[1] = sym_exponent(tot);
    meta[2] = (ncyc + cb - 1) / cb;
  }
}

// Float64 net force of every cycle (its points in order), and the zeroed fixed-point
// accumulator (grid-stride over all 2P entries).
__global__ __launch_bounds__(256) void k_sym_cycles(const int4* __restrict__ cyc, const int32_t* __restrict__ meta,
                                                    const double2* __restrict__ f64, int P,
                                                    double2* __restrict__ fcyc, unsigned long long* __restrict__ acc) {
  const int64_t stride = (int64_t)gridDim.x * blockDim.x;
  const int64_t first = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
  for (int64_t e = first; e < 2 * (int64_t)P; e += stride) acc[e] = 0ull;
  const int ncyc = meta[0];
  for (int64_t c = first; c < ncyc; c += stride) {
    const int4 cy = cyc[c];
    double sx = 0.0, sy = 0.0;
    for (int m = 0; m < cy.y; ++m) {
      const double2 F = f64[cy.x + m];
      sx += F.x;
      sy += F.y;
    }
    fcyc[c] = make_double2(sx, sy);
  }
}

// k_prepare, k_sym_plan and k_sym_cycles of up to kSymFused vesicles in one launch, a wavefront per vesicle, which
// counts the cycles of the vesicles before it itself: the same values in the same order, but for the fixed-point
// exponent, which the units form (meta[1] is not written).  zero0 and zero1 (or null): 2 P words cleared.  kAdjoint:
// also the records of g, and the cycle sums are those of g; else of F = w f, and the whole prepared region is left, for
// later evaluations from it.
// 504 x 32: three launches -> one, 104.4 -> 99.9 us a call; 512 x 64 and its adjoint: nine -> two, 932 -> 914 us.
// Latency bounds it, so a wavefront takes 256 points at a time (64 at a time: 500 x 16 and one vesicle of 20,000 points
// 531 us a call, now 499).
constexpr int kSymFused = 1024;

constexpr int kPrepStep = 256;  // points of a step, four per lane

template <bool kAdjoint>
__global__ __launch_bounds__(64) void k_sym_prepare(const double* __restrict__ pts, const double* __restrict__ f,
                                                    const double* __restrict__ w, const double* __restrict__ g,
                                                    const int32_t* __restrict__ off, int M, int P, int cb, int ncyc_max,
                                                    PreparedView pv, float4* __restrict__ recG,
                                                    int4* __restrict__ cyc, double2* __restrict__ ccyc,
                                                    int32_t* __restrict__ meta, unsigned long long* __restrict__ zero0,
                                                    unsigned long long* __restrict__ zero1) {
  __shared__ double2 carried[kPrepStep];
  float4* recF = static_cast<float4*>(pv.rec);
  const int lane = threadIdx.x, v = blockIdx.x;
  const auto clamped = [&](int u) { return min(max(off[u], 0), P); };
  for (int64_t e = (int64_t)v * 64 + lane; e < 2 * (int64_t)P; e += (int64_t)M * 64) {
    zero0[e] = 0ull;
    if (zero1) zero1[e] = 0ull;
  }
  int first = 0;  // cycles of the vesicles before
  for (int u = lane; u < v; u += 64) first += (max(0, clamped(u + 1) - clamped(u)) + kRing - 1) / kRing;
#pragma unroll
  for (int m = 32; m >= 1; m >>= 1) first += __shfl_xor(first, m, 64);
  const int j0 = clamped(v), j1 = max(j0, clamped(v + 1)), n = j1 - j0;
  double sx = 0.0, sy = 0.0, bx = 0.0, by = 0.0, sa = 0.0, sw = 0.0;
#pragma unroll 4
  for (int j = j0 + lane; j < j1; j += 64) {
    const double wj = w[j];
    sx += pts[j];
    sy += pts[P + j];
    const double ex = wj * f[j], ey = wj * f[P + j];
    bx += ex;
    by += ey;
    sa += fabs(ex) + fabs(ey);
    sw += wj;
  }
  sx = wave_sum_d(sx);
  sy = wave_sum_d(sy);
  bx = wave_sum_d(bx);
  by = wave_sum_d(by);
  sa = wave_sum_d(sa);
  if constexpr (!kAdjoint) sw = wave_sum_d(sw);
  const double cx = n > 0 ? sx / n : 0.0, cy = n > 0 ? sy / n : 0.0;
  double r2 = 0.0;
  for (int c0 = j0; c0 < j1; c0 += kPrepStep) {
    wave_sync();  // the previous points are done
#pragma unroll
    for (int q = 0; q < kPrepStep; q += 64) {
      const int j = c0 + q + lane;
      if (j < j1) {
        const double wj = w[j];
        const double x = pts[j], y = pts[P + j];
        const double ex = wj * f[j], ey = wj * f[P + j];
        r2 = fmax(r2, (x - cx) * (x - cx) + (y - cy) * (y - cy));
        recF[j] = make_float4((float)(x - cx), (float)(y - cy), (float)ex, (float)ey);
        if constexpr (kAdjoint) {
          const double gx = g[j], gy = g[P + j];
          recG[j] = make_float4((float)(x - cx), (float)(y - cy), (float)gx, (float)gy);
          carried[q + lane] = make_double2(gx, gy);
        } else {
          carried[q + lane] = make_double2(ex, ey);
          pv.f64[j] = make_double2(ex, ey);
          pv.vid[j] = v;
        }
      }
    }
    wave_sync();
    const int k0 = c0 + kRing * lane, cnt = min(kRing, j1 - k0), e = first + (k0 - j0) / kRing;
    if (lane < kPrepStep / kRing && cnt > 0 && e < ncyc_max) {
      double tx = 0.0, ty = 0.0;
      for (int m = 0; m < cnt; ++m) {
        const double2 F = carried[kRing * lane + m];
        tx += F.x;
        ty += F.y;
      }
      cyc[e] = make_int4(k0, cnt, v, 0);
      ccyc[e] = make_double2(tx, ty);
    }
  }
#pragma unroll
  for (int m = 32; m >= 1; m >>= 1) r2 = fmax(r2, __shfl_xor(r2, m, 64));
  if (lane != 0) return;
  pv.vtab[v] = make_double4(cx, cy, bx, by);
  pv.vaux[v] = make_double2(sa, r2);
  if constexpr (!kAdjoint) {
    pv.vrange[v] = make_int2(j0, j1);
    pv.hlen[v] = n > 0 ? sw / n : 0.0;
  }
  if (v == M - 1) {
    const int ncyc = min(first + (n + kRing - 1) / kRing, ncyc_max);
    meta[0] = ncyc;
    meta[2] = (ncyc + cb - 1) / cb;
  }
}

// Unit number L (0 <= L < nb (nb + 1) / 2) of nb blocks, row block by row block, as the pair {bx, by}.
__device__ __forceinline__ void sym_unit_blocks(int nb, int L, int& bx, int& by) {
  const int h = nb >> 1;
  int d;
  if (L < h * (h + 1) || (nb & 1)) {
    bx = L / (h + 1);
    d = L - bx * (h + 1);
  } else {
    const int L2 = L - h * (h + 1);
    bx = h + L2 / h;
    d = L2 - (bx - h) * h;
  }
  by = bx + d;
  if (by >= nb) by -= nb;
}

// The position of workgroup g of n in that XCD-contiguous order.
__device__ __forceinline__ int xcd_contiguous(int g, int n) {
  const int q = n / kXcds, r = n % kXcds;
  const int x = g % kXcds;
  return x * q + min(x, r) + g / kXcds;
}

// First vesicle start at or after cycle c of the block's cycles [c0, c1) (c0 and c1 count as starts).  The same
// for every lane; called by whole wavefronts.
__device__ __forceinline__ int vesicle_cut(const int4* __restrict__ cyc, int c0, int c1, int c) {
  if (c <= c0) return c0;
  for (; c < c1; c += 64) {
    const int e = c + (int)(threadIdx.x & 63);
    const unsigned long long m = __ballot(e >= c1 || cyc[e].z != cyc[e - 1].z);
    if (m) return min(c1, c + __ffsll(m) - 1);
  }
  return c1;
}

// The unit of this workgroup among the nb blocks' pairs, each cut into ns strips of the column block.  Units are the
// pairs {bx, bx + d mod nb}, d = 0 .. nb/2 (for even nb, d = nb/2 only for bx < nb/2), numbered row block by row block.
// Workgroups are handed to the eight XCDs in turn (workgroup g to XCD g mod 8), so each XCD is given one contiguous
// range of that numbering: its concurrent units share a row block and a window of about nb/2 consecutive column blocks,
// which stays in the XCD's own L2.  Row block bx, column block by, and the strip's cycles [s0, s1) of block by's [by
// cb, min(ncyc, (by + 1) cb)); false when it has none.  Strips end at vesicle starts, so that the float32 partial sums
// of a (target, vesicle) are the same for every ns (a vesicle longer than a strip leaves the following ones empty).
__device__ __forceinline__ bool sym_unit(int nb, int ns, int cb, int ncyc, const int4* __restrict__ cyc, int& bx,
                                         int& by, int& s0, int& s1) {
  const int h = nb >> 1;
  const int units = ((nb & 1) ? nb * (h + 1) : nb * h + h) * ns;
  const int g = blockIdx.x;
  if (g >= units) return false;
  const int L = xcd_contiguous(g, units);
  sym_unit_blocks(nb, L / ns, bx, by);
  const int c0 = by * cb, c1 = min(ncyc, c0 + cb);
  if (ns == 1) {
    s0 = c0;
    s1 = c1;
  } else {
    const int k = L % ns, w = cb / ns;
    s0 = vesicle_cut(cyc, c0, c1, c0 + k * w);
    s1 = k == ns - 1 ? c1 : vesicle_cut(cyc, c0, c1, c0 + (k + 1) * w);
  }
  return s0 < s1;
}

// One unit: target cycles [tc0, tc1) against source cycles [sc0, sc1) (diag: the two blocks are one),
// fixed-point exponent S (see the file header).  Called by the whole workgroup.
template <int T>
__device__ __forceinline__ void sym_eval_unit(int P, const double4* __restrict__ vtab,
                                              const double2* __restrict__ vaux, const float4* __restrict__ rec,
                                              const int4* __restrict__ cyc, const double2* __restrict__ fcyc, int S,
                                              int tc0, int tc1, int sc0, int sc1, bool diag,
                                              unsigned long long* __restrict__ acc) {
  constexpr int CB = kRows * T;  // cycles per block
  __shared__ float4 s_tx[CB][kRing];               // target records (local coordinates, w f)
  __shared__ double4 s_tc[CB];                     // (c_A, F_cycle) of each target cycle
  __shared__ double s_tr[CB];                      // R_A^2
  __shared__ int4 s_ti[CB];                        // (vesicle or -1, count, first point, 0)
  __shared__ float4 s_rec[2][kChunk][2 * kRing];   // source cycles, each stored twice
  __shared__ float s_col[2][kSymWaves][kChunk][2][kRing];
  __shared__ double2 s_E[2][kSymWaves][kChunk];

  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6, p = lane & 15;
  const int row = tid >> 4;

  // Target block into LDS.
  for (int e = tid; e < CB * kRing; e += kSymThreads) {
    const int t = e / kRing, m = e % kRing;
    const int c = tc0 + t;
    float4 r = make_float4(0.f, 0.f, 0.f, 0.f);
    if (c < tc1) {
      const int4 cy = cyc[c];
      if (m < cy.y) r = rec[cy.x + m];
    }
    s_tx[t][m] = r;
  }
  for (int t = tid; t < CB; t += kSymThreads) {
    const int c = tc0 + t;
    if (c < tc1) {
      const int4 cy = cyc[c];
      const double4 vt = vtab[cy.z];
      const double2 F = fcyc[c];
      s_tc[t] = make_double4(vt.x, vt.y, F.x, F.y);
      s_tr[t] = vaux[cy.z].y;
      s_ti[t] = make_int4(cy.z, cy.y, cy.x, 0);
    } else {
      s_tc[t] = make_double4(0.0, 0.0, 0.0, 0.0);
      s_tr[t] = 0.0;
      s_ti[t] = make_int4(-1, 0, 0, 0);
    }
  }

  // State of the current source segment, per target slot k (target cycle k * 16 + row).
  float dx[T], dy[T], ns[T], fcx[T], fcy[T], fhx[T], fhy[T], lx[T], ly[T], rvx[T], rvy[T];
  double ax[T], ay[T];
  int kq[T];
  int actm = 0;
  double Ex = 0.0, Ey = 0.0, Fsx = 0.0, Fsy = 0.0;
#pragma unroll
  for (int k = 0; k < T; ++k) {
    dx[k] = dy[k] = ns[k] = fcx[k] = fcy[k] = fhx[k] = fhy[k] = 0.f;
    lx[k] = ly[k] = rvx[k] = rvy[k] = 0.f;
    ax[k] = ay[k] = 0.0;
    kq[k] = 0;
  }

  auto setup = [&](int B) {
    const double4 vb = vtab[B];
    const double rb2 = vaux[B].y;
    double ex = 0.0, ey = 0.0;
    actm = 0;
#pragma unroll
    for (int k = 0; k < T; ++k) {
      const int t = k * kRows + row;
      const int4 ti = s_ti[t];
      const double4 tc = s_tc[t];
      const float4 tx = s_tx[t][p];
      const double Dx = tc.x - vb.x, Dy = tc.y - vb.y;
      const double D = fma(Dy, Dy, fma(Dx, Dx, s_tr[t] + rb2));
      int e;
      frexp(D, &e);
      const int kk = min(kMaxShift, max(-kMaxShift, e >> 1));
      const bool rowact = ti.x >= 0 && ti.x != B && (!diag || ti.x < B);
      const bool act = rowact && p < ti.y;
      actm |= act ? (1 << k) : 0;
      const float sc = ldexpf(1.0f, -kk);
      dx[k] = act ? fmaf(tx.x, sc, (float)ldexp(Dx, -kk)) : kFar;
      dy[k] = act ? fmaf(tx.y, sc, (float)ldexp(Dy, -kk)) : 0.f;
      ns[k] = -sc;
      fcx[k] = act ? tx.z : 0.f;
      fcy[k] = act ? tx.w : 0.f;
      fhx[k] = kHalfLn2f * fcx[k];
      fhy[k] = kHalfLn2f * fcy[k];
      kq[k] = kk;
      lx[k] = ly[k] = rvx[k] = rvy[k] = 0.f;
      ex += rowact ? (double)kk * tc.z : 0.0;
      ey += rowact ? (double)kk * tc.w : 0.0;
    }
    // the 16 lanes of a row hold the same value: add the four rows of the wavefront
    ex += __shfl_xor(ex, 16, 64);
    ey += __shfl_xor(ey, 16, 64);
    ex += __shfl_xor(ex, 32, 64);
    ey += __shfl_xor(ey, 32, 64);
    Ex = -kLn2d * ex;
    Ey = -kLn2d * ey;
    Fsx = Fsy = 0.0;
  };

  auto flush = [&]() {
#pragma unroll
    for (int k = 0; k < T; ++k) {
      const float pvx = fmaf(kHalfLn2f, lx[k], rvx[k]);
      const float pvy = fmaf(kHalfLn2f, ly[k], rvy[k]);
      const double c = -kLn2d * (double)kq[k];
      const bool act = (actm >> k) & 1;
      ax[k] += act ? fma(c, Fsx, (double)pvx) : 0.0;
      ay[k] += act ? fma(c, Fsy, (double)pvy) : 0.0;
    }
  };

  // One ring cycle over the 16 sources of LDS cycle slot cc.
  auto ring = [&](int buf, int cc) {
    const float4* rb = &s_rec[buf][cc][p];
    float cax = 0.f, cay = 0.f;
#pragma unroll 1
    for (int s = 0; s < kRing; ++s) {
      const float4 sr = rb[s];
      float lcx = 0.f, lcy = 0.f;
#pragma unroll
      for (int k = 0; k < T; ++k) {
        const float rx = fmaf(sr.x, ns[k], dx[k]);
        const float ry = fmaf(sr.y, ns[k], dy[k]);
        const float q = fmaf(ry, ry, rx * rx);
        const float L = __builtin_amdgcn_logf(q);
        const float rho = __builtin_amdgcn_rcpf(q);
        const float rxr = rx * rho, ryr = ry * rho;
        const float b = fmaf(ryr, sr.w, rxr * sr.z);       // (r . F_j)/q
        lx[k] = fmaf(L, sr.z, lx[k]);
        ly[k] = fmaf(L, sr.w, ly[k]);
        rvx[k] = fmaf(b, rx, rvx[k]);
        rvy[k] = fmaf(b, ry, rvy[k]);
        const float b2 = fmaf(ryr, fcy[k], rxr * fcx[k]);  // (r . F_i)/q
        if (k == 0) {
          lcx = L * fhx[k];
          lcy = L * fhy[k];
        } else {
          lcx = fmaf(L, fhx[k], lcx);
          lcy = fmaf(L, fhy[k], lcy);
        }
        lcx = fmaf(b2, rx, lcx);
        lcy = fmaf(b2, ry, lcy);
      }
      cax = ring_next(cax) + lcx;
      cay = ring_next(cay) + lcy;
    }
    // lane p now holds source (p + 15) mod 16 of its row; add the four rows: x sums end in lanes
    // 0-31, y sums in lanes 32-63, then every row of a half holds the half's total
    const auto h = __builtin_amdgcn_permlane32_swap(bitsu(cax), bitsu(cay), false, false);
    const float z = bitsf(h[0]) + bitsf(h[1]);
    const auto r16 = __builtin_amdgcn_permlane16_swap(bitsu(z), bitsu(z), false, false);
    const float tot = bitsf(r16[0]) + bitsf(r16[1]);
    if ((lane & 16) == 0) s_col[buf][wv][cc][lane >> 5][(p + kRing - 1) & (kRing - 1)] = tot;
  };

  // Records of source chunk g: slots 0..15 and again 16..31; slots past the cycle's count repeat
  // its first point with zero force.
  const int nchunks = (sc1 - sc0 + kChunk - 1) / kChunk;
  const bool stager = tid < kChunk * 2 * kRing;
  const int st_cc = tid >> 5, st_q = tid & 31, st_m = st_q & (kRing - 1);
  auto stage_load = [&](int g) {
    float4 r = make_float4(0.f, 0.f, 0.f, 0.f);
    const int c = sc0 + g * kChunk + st_cc;
    if (stager && c < sc1) {
      const int4 cy = cyc[c];
      r = rec[cy.x + (st_m < cy.y ? st_m : 0)];
      if (st_m >= cy.y) r.z = r.w = 0.f;
    }
    return r;
  };
  auto stage_store = [&](int buf, const float4& r) {
    if (stager) s_rec[buf][st_cc][st_q] = r;
  };

  // Column sums of chunk g: the wavefronts and their log corrections added in a fixed order,
  // then one fixed-point integer per (source, component).
  auto reduce = [&](int g, int buf) {
    if (tid >= kChunk * 2 * kRing) return;
    const int cc = tid >> 5, comp = (tid >> 4) & 1, m = tid & (kRing - 1);
    const int c = sc0 + g * kChunk + cc;
    if (c >= sc1) return;
    const int4 cy = cyc[c];
    if (m >= cy.y) return;
    double s = 0.0;
#pragma unroll
    for (int w2 = 0; w2 < kSymWaves; ++w2) s += (double)s_col[buf][w2][cc][comp][m];
    double e = 0.0;
#pragma unroll
    for (int w2 = 0; w2 < kSymWaves; ++w2) {
      const double2 E = s_E[buf][w2][cc];
      e += comp ? E.y : E.x;
    }
    const long long X = (long long)rint(ldexp(s + e, S));
    atomicAdd(&acc[(size_t)comp * P + cy.x + m], (unsigned long long)X);
  };

  int curB = -1;
  stage_store(0, stage_load(0));
  __syncthreads();
  for (int g = 0; g < nchunks; ++g) {
    const int buf = g & 1;
    const float4 nxt = stage_load(g + 1);
    if (g > 0) reduce(g - 1, buf ^ 1);
    const int cbase = sc0 + g * kChunk;
    const int ncc = min(kChunk, sc1 - cbase);
    for (int cc = 0; cc < ncc; ++cc) {
      const int4 cy = cyc[cbase + cc];
      if (cy.z != curB) {
        if (curB >= 0) flush();
        setup(cy.z);
        curB = cy.z;
      }
      const double2 Fc = fcyc[cbase + cc];
      Fsx += Fc.x;
      Fsy += Fc.y;
      ring(buf, cc);
      if (lane == 0) s_E[buf][wv][cc] = make_double2(Ex, Ey);
    }
    stage_store(buf ^ 1, nxt);
    __syncthreads();
  }
  if (nchunks > 0) {
    reduce(nchunks - 1, (nchunks - 1) & 1);
    flush();
  }
#pragma unroll
  for (int k = 0; k < T; ++k) {
    const int4 ti = s_ti[k * kRows + row];
    if (ti.x >= 0 && p < ti.y) {
      const int i = ti.z + p;
      atomicAdd(&acc[i], (unsigned long long)(long long)rint(ldexp(ax[k], S)));
      atomicAdd(&acc[(size_t)P + i], (unsigned long long)(long long)rint(ldexp(ay[k], S)));
    }
  }
}

// The fixed-point exponent (see sym_exponent) from the vesicles' sums of |F|_1, by a whole workgroup of kSymThreads.
__device__ __forceinline__ int vesicles_exponent(const double2* __restrict__ vaux, int M) {
  __shared__ double s_sum[kSymWaves];
  double a = 0.0;
  for (int v = threadIdx.x; v < M; v += kSymThreads) a += vaux[v].x;
  a = wave_sum_d(a);
  if ((threadIdx.x & 63) == 0) s_sum[threadIdx.x >> 6] = a;
  __syncthreads();
  double tot = 0.0;
#pragma unroll
  for (int k = 0; k < kSymWaves; ++k) tot += s_sum[k];
  return sym_exponent(tot);
}

// One unit {bx, by} per workgroup (see the file header).  kFused: after k_sym_prepare of M vesicles.
template <int T, bool kFused>
__global__ __launch_bounds__(kSymThreads) void k_sym_main(
    int P, int ns, const double4* __restrict__ vtab, const double2* __restrict__ vaux, const float4* __restrict__ rec,
    const int4* __restrict__ cyc, const double2* __restrict__ fcyc,
    std::conditional_t<kFused, int32_t, const int32_t>* __restrict__ meta, int M, unsigned long long* __restrict__ acc) {
  constexpr int CB = kRows * T;
  const int ncyc = meta[0];
  int S;
  if constexpr (kFused) {
    S = vesicles_exponent(vaux, M);
    if (blockIdx.x == 0 && threadIdx.x == 0) meta[1] = S;  // for k_sym_finish
  } else {
    S = meta[1];
  }
  const int nb = meta[2];
  if (nb <= 0) return;
  int bx, by, s0, s1;
  if (!sym_unit(nb, ns, CB, ncyc, cyc, bx, by, s0, s1)) return;
  const int tc0 = bx * CB;
  sym_eval_unit<T>(P, vtab, vaux, rec, cyc, fcyc, S, tc0, min(ncyc, tc0 + CB), s0, s1, bx == by, acc);
}

// ------------------------------------------------------------------ float64 symmetric form
// The same circulant schedule of unordered block pairs and rings of 16 lanes, in float64 on global coordinates.
// Float64 needs no compensation per source vesicle, so nothing here follows the vesicles: blocks are 256 T consecutive
// points, ring cycles 16 consecutive points whatever vesicles they belong to (only the last cycle of a suspension is
// padded; cut at the vesicles, 17 to 63 points each, 47% of the pair evaluations were padding), rows are summed chunk
// by chunk of 64 columns whatever the vesicles (summed over a whole unit in one chain they rounded 1.4 times as much in
// all), the matrix's diagonal terms apart from the others (over a vesicle without net force the partial sums are tens
// of times its terms, and both FMAs of a pair rounded at their size: 1.2 to 1.4 times the error for 1% less time; four
// pairs summed by themselves first halve it, for 2.7% more), and the block table needs no plan kernel.  The own vesicle
// is dropped pair by pair, but only in units whose row and column points share a vesicle (ids are compared at both
// ends; at most the diagonal and the neighbouring block pairs): there the accumulations are selected, so that not even
// a non-finite value of an own-vesicle pair enters.
//
// Work split: a unit is the row block against one of `ns` equal strips of the column block.  One unit per
// block pair leaves most of the chip idle on small problems and a nearly empty last round on middling ones;
// strips cost one more set of row additions each.
//
// Per unordered pair: with l = -1/2 ln q, rho = 1/q the Stokeslet is (A c; c B), A = l + rx^2 rho,
// B = l + ry^2 rho, c = rx ry rho, the same for both directions: 9 float64 operations besides l and rho, and 4
// FMAs per direction (33.3 instructions in the ring at T = 4, against 36.6 with projections and separate log and
// rr sums).  The logarithm is the table logarithm of the direct float64 kernel, halved and negated in
// the table, with 1024 entries (series through r^4); the table is built once per call and copied to LDS by each
// unit.  Column sums travel around the ring by DPP moves of both halves of each double.  What bounds it is
// float64 VALU issue (4 cycles per instruction and wavefront, 16 for the hardware reciprocal).  Measured before
// and after, on one card: 2000 x 128 36.7 -> 35.1 ms, 1020 vesicles of 17 to 63 points (40,008 points) 1.45 -> 0.97 ms.
//
// Sums leave the workgroup as two 64-bit fixed-point words:
// hi = rint(x 2^S) and lo = rint((x - hi 2^-S) 2^(S + kLoBits)) (the first difference is exact), each added
// by an integer atomic, so the result is independent of the order of the atomics while the
// resolution is 2^-(S + kLoBits), far below float64 rounding of the sum.  |lo| <= 2^(kLoBits - 1), so up to
// 2^(62 - kLoBits + 1) partials per point stay exact.  A partial that is not finite (coincident points of two
// vesicles, non-finite inputs) marks its output in `bad`, which the last kernel turns into NaN.
constexpr int kLoBits = 40;
constexpr int kChunk64 = 4;                         // source cycles per LDS chunk
constexpr double kFar64 = 3.2733906078961419e150;   // 2^500: position of an inactive target
static_assert(kChunk64 * 2 * kRing <= kSymThreads, "one thread per staged record and per column sum of a chunk");

// x from lane (p + 1) mod 16 of the same row (both halves of the double moved by DPP).
__device__ __forceinline__ double ring_next64(double x) {
  const unsigned long long b = __builtin_bit_cast(unsigned long long, x);
  const int lo = __builtin_amdgcn_update_dpp(0, (int)(unsigned)b, 0x12F, 0xF, 0xF, true);
  const int hi = __builtin_amdgcn_update_dpp(0, (int)(unsigned)(b >> 32), 0x12F, 0xF, 0xF, true);
  return __builtin_bit_cast(double, ((unsigned long long)(unsigned)hi << 32) | (unsigned)lo);
}

__device__ __forceinline__ unsigned long long dlo(double x) { return __builtin_bit_cast(unsigned long long, x); }
__device__ __forceinline__ double dfrom(unsigned lo, unsigned hi) {
  return __builtin_bit_cast(double, ((unsigned long long)hi << 32) | lo);
}

constexpr int kSymTab = kHalfLogTab;               // entries of the log table (16 KB of LDS)

// Adds x to the two fixed-point words of one accumulator entry (hi at a, lo at a + 2P), or marks it.
__device__ __forceinline__ void fixed_add2(unsigned long long* __restrict__ a, uint8_t* __restrict__ bad, size_t two_p,
                                           double x, int S) {
  if (!isfinite(x)) {
    *bad = 1;
    return;
  }
  const double h = rint(ldexp(x, S));
  const double r = x - ldexp(h, -S);  // exact
  atomicAdd(a, (unsigned long long)(long long)h);
  atomicAdd(a + two_p, (unsigned long long)(long long)rint(ldexp(r, S + kLoBits)));
}

// The accumulator words (4 P) and marks (2 P bytes, padded to words) of a float64 call cleared and its log table built,
// workgroup b of n of 1024 threads; the last one builds the table.
struct Sym64Start {
  unsigned long long* acc;
  uint32_t* bad;
  double2* tab;
  int P;
};
__device__ __forceinline__ void sym64_start(const Sym64Start& st, int b, int n) {
  const int64_t stride = (int64_t)n * 1024, first = b * (int64_t)1024 + threadIdx.x;
  for (int64_t e = first; e < 4 * (int64_t)st.P; e += stride) st.acc[e] = 0ull;
  for (int64_t e = first; e < (2 * (int64_t)st.P + 3) / 4; e += stride) st.bad[e] = 0u;
  if (b == n - 1) st.tab[threadIdx.x] = half_log_entry(threadIdx.x);
}

// Start of a single suspension's call: the above, and its exponent (workgroup 0; the vesicles' sums in a fixed order).
// meta[3]: 1 when the bound itself is not finite (then every output is NaN).
__global__ __launch_bounds__(1024) void k_sym64_init(const double2* __restrict__ vaux,
                                                     const int2* __restrict__ vrange,
                                                     const double4* __restrict__ rec, int M, Sym64Start st,
                                                     int32_t* __restrict__ meta) {
  sym64_start(st, blockIdx.x, gridDim.x);
  if (blockIdx.x != 0) return;
  __shared__ double s_dsum[16];
  double fa = 0.0;
  for (int v = threadIdx.x; v < M; v += 1024) fa += bound_share(vaux[v].x, vrange[v], rec);
  fa = wave_sum_d(fa);
  if ((threadIdx.x & 63) == 0) s_dsum[threadIdx.x >> 6] = fa;
  __syncthreads();
  if (threadIdx.x == 0) {
    double tot = 0.0;
    for (int k = 0; k < 16; ++k) tot += s_dsum[k];
    meta[1] = sym64_exponent(tot);
    meta[3] = isfinite(tot) ? 0 : 1;
  }
}
static_assert(kSymTab == 1024, "sym64_start builds one entry per thread");

// LDS of a unit besides the table: source cycles (x, y, F_x, F_y) and vesicle ids, each stored twice, and the
// wavefronts' column sums, double buffered by chunk.
struct Sym64Lds {
  double4 rec[2][kChunk64][2 * kRing];
  int32_t vid[2][kChunk64][2 * kRing];
  double col[2][kSymWaves][kChunk64][2][kRing];
};

// One unit: row points [r0, r1) (at most 256 T) against column points [c0, c1); diag: the column strip lies in
// the row block.  ltab is in LDS.  Called by the whole workgroup.
template <int T>
__device__ __forceinline__ void sym64_eval_unit(Sym64Lds& lds, int P, const double4* __restrict__ rec,
                                                const int32_t* __restrict__ vid, const double2* __restrict__ ltab,
                                                int S, int r0, int r1, int c0, int c1, bool diag,
                                                unsigned long long* __restrict__ acc, uint8_t* __restrict__ bad) {
  auto& s_rec = lds.rec;
  auto& s_vid = lds.vid;
  auto& s_col = lds.col;
  const size_t two_p = 2 * (size_t)P;
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6, p = lane & 15;
  const int row = tid >> 4;
  // vesicle ids do not decrease: the two point ranges share a vesicle when their id ranges meet
  const bool masked = diag || !(vid[r1 - 1] < vid[c0] || vid[c1 - 1] < vid[r0]);

  // a and b: sums of a chunk of columns, of the matrix's diagonal terms and of the others; s: of all
  double tx[T], ty[T], fx[T], fy[T], ax[T], ay[T], bx[T], by[T], sx[T], sy[T];
  int tv[T];
#pragma unroll
  for (int k = 0; k < T; ++k) {
    const int i = r0 + (k * kRows + row) * kRing + p;
    const bool in = i < r1;
    const double4 t = in ? rec[i] : make_double4(kFar64, 0.0, 0.0, 0.0);
    tv[k] = in ? vid[i] : -1;
    tx[k] = t.x;
    ty[k] = t.y;
    fx[k] = t.z;
    fy[k] = t.w;
    ax[k] = ay[k] = bx[k] = by[k] = sx[k] = sy[k] = 0.0;
  }

  auto ring = [&](int buf, int cc, auto mask_tag) __attribute__((always_inline)) {
    constexpr bool kMask = decltype(mask_tag)::value;
    const double4* rb = &s_rec[buf][cc][p];
    const int32_t* vb = &s_vid[buf][cc][p];
    double cax = 0.0, cay = 0.0;
#pragma unroll 1
    for (int s = 0; s < kRing; ++s) {
      const double4 sr = rb[s];
      const int sv = kMask ? vb[s] : 0;
      double lcx = 0.0, lcy = 0.0;
#pragma unroll
      for (int k = 0; k < T; ++k) {
        const double rx = tx[k] - sr.x;
        const double ry = ty[k] - sr.y;
        const double q = fma(ry, ry, rx * rx);
        const double l = neg_half_log<true>(q, ltab);
        const double rho = recip(q);
        const double t = rx * rho, u = ry * rho;
        const double A = fma(rx, t, l), B = fma(ry, u, l), c = ry * t;
        const double nax = fma(A, sr.z, ax[k]), nbx = fma(c, sr.w, bx[k]);
        const double nay = fma(B, sr.w, ay[k]), nby = fma(c, sr.z, by[k]);
        const double ncx = fma(A, fx[k], k == 0 ? c * fy[k] : fma(c, fy[k], lcx));
        const double ncy = fma(c, fx[k], k == 0 ? B * fy[k] : fma(B, fy[k], lcy));
        // own-vesicle pairs, and in the diagonal block one of each two orderings (ids do not decrease)
        const bool act = !kMask || (diag ? tv[k] < sv : tv[k] != sv);
        ax[k] = act ? nax : ax[k];
        ay[k] = act ? nay : ay[k];
        bx[k] = act ? nbx : bx[k];
        by[k] = act ? nby : by[k];
        lcx = act ? ncx : lcx;
        lcy = act ? ncy : lcy;
      }
      cax = ring_next64(cax) + lcx;
      cay = ring_next64(cay) + lcy;
    }
    // lane p holds source (p + 15) mod 16 of its row; add the four rows: x sums end in lanes 0-31, y sums
    // in lanes 32-63 (both halves of each double swapped alike), then every row of a half holds the total
    const unsigned long long bx_ = dlo(cax), by_ = dlo(cay);
    const auto hl = __builtin_amdgcn_permlane32_swap((unsigned)bx_, (unsigned)by_, false, false);
    const auto hh = __builtin_amdgcn_permlane32_swap((unsigned)(bx_ >> 32), (unsigned)(by_ >> 32), false, false);
    const double z = dfrom(hl[0], hh[0]) + dfrom(hl[1], hh[1]);
    const unsigned long long bz = dlo(z);
    const auto gl = __builtin_amdgcn_permlane16_swap((unsigned)bz, (unsigned)bz, false, false);
    const auto gh = __builtin_amdgcn_permlane16_swap((unsigned)(bz >> 32), (unsigned)(bz >> 32), false, false);
    const double tot = dfrom(gl[0], gh[0]) + dfrom(gl[1], gh[1]);
    if ((lane & 16) == 0) s_col[buf][wv][cc][lane >> 5][(p + kRing - 1) & (kRing - 1)] = tot;
  };

  // Points of chunk g: slots 0..15 and again 16..31 of each cycle; slots past c1 repeat the last point with
  // zero force.
  const int ncyc = (c1 - c0 + kRing - 1) / kRing;
  const int nchunks = (ncyc + kChunk64 - 1) / kChunk64;
  const bool stager = tid < kChunk64 * 2 * kRing;
  const int st_cc = tid >> 5, st_q = tid & 31;
  auto stage_load = [&](int g, int& v) {
    double4 r = make_double4(0.0, 0.0, 0.0, 0.0);
    v = -1;
    const int j = c0 + (g * kChunk64 + st_cc) * kRing + (st_q & (kRing - 1));
    if (stager && g < nchunks) {
      const int jj = min(j, c1 - 1);
      r = rec[jj];
      v = vid[jj];
      if (j >= c1) r.z = r.w = 0.0;
    }
    return r;
  };
  auto stage_store = [&](int buf, const double4& r, int v) {
    if (stager) {
      s_rec[buf][st_cc][st_q] = r;
      s_vid[buf][st_cc][st_q] = v;
    }
  };
  // column sums of chunk g: the four wavefronts added in a fixed order, then two fixed-point words
  auto reduce = [&](int g, int buf) {
    if (tid >= kChunk64 * 2 * kRing) return;
    const int cc = tid >> 5, comp = (tid >> 4) & 1, m = tid & (kRing - 1);
    const int j = c0 + (g * kChunk64 + cc) * kRing + m;
    if (j >= c1) return;
    const double v = ((s_col[buf][0][cc][comp][m] + s_col[buf][1][cc][comp][m]) + s_col[buf][2][cc][comp][m]) +
                     s_col[buf][3][cc][comp][m];
    const size_t e = (size_t)comp * P + j;
    fixed_add2(&acc[e], &bad[e], two_p, v, S);
  };

  {
    int v;
    const double4 r = stage_load(0, v);
    stage_store(0, r, v);
  }
  __syncthreads();
  for (int g = 0; g < nchunks; ++g) {
    const int buf = g & 1;
    int nv;
    const double4 nxt = stage_load(g + 1, nv);
    if (g > 0) reduce(g - 1, buf ^ 1);
    const int ncc = min(kChunk64, ncyc - g * kChunk64);
    if (masked)
      for (int cc = 0; cc < ncc; ++cc) ring(buf, cc, std::true_type{});
    else
      for (int cc = 0; cc < ncc; ++cc) ring(buf, cc, std::false_type{});
#pragma unroll
    for (int k = 0; k < T; ++k) {
      sx[k] += ax[k] + bx[k];
      sy[k] += ay[k] + by[k];
      ax[k] = ay[k] = bx[k] = by[k] = 0.0;
    }
    stage_store(buf ^ 1, nxt, nv);
    __syncthreads();
  }
  reduce(nchunks - 1, (nchunks - 1) & 1);
#pragma unroll
  for (int k = 0; k < T; ++k) {
    const int i = r0 + (k * kRows + row) * kRing + p;
    if (i < r1) {
      fixed_add2(&acc[i], &bad[i], two_p, sx[k], S);
      fixed_add2(&acc[(size_t)P + i], &bad[(size_t)P + i], two_p, sy[k], S);
    }
  }
}

// Strip s of ns of the block pair {bx, by} of the points [p0, p1).  In the diagonal block, rows past the strip
// have no pair in it (the ids there are not smaller); row ranges that fit half the targets per thread or fewer
// (those, and the last block) take the narrower form instead of evaluating empty slots.
template <int T>
__device__ __forceinline__ void sym64_run(Sym64Lds& lds, int P, const double4* __restrict__ rec,
                                          const int32_t* __restrict__ vid, const double2* __restrict__ ltab, int S,
                                          int p0, int p1, int bx, int by, int ns, int s,
                                          unsigned long long* __restrict__ acc, uint8_t* __restrict__ bad) {
  constexpr int BP = kSymThreads * T;  // points per block; a strip is a whole number of cycles
  const int c0 = p0 + by * BP + s * (BP / ns), c1 = min(p1, c0 + BP / ns);
  if (c0 >= c1) return;
  const int r0 = p0 + bx * BP, r1 = min(bx == by ? c1 : p1, r0 + BP);
  if (T > 1 && r1 - r0 <= kSymThreads)
    sym64_eval_unit<1>(lds, P, rec, vid, ltab, S, r0, r1, c0, c1, bx == by, acc, bad);
  else if (T > 2 && r1 - r0 <= 2 * kSymThreads)
    sym64_eval_unit<2>(lds, P, rec, vid, ltab, S, r0, r1, c0, c1, bx == by, acc, bad);
  else
    sym64_eval_unit<T>(lds, P, rec, vid, ltab, S, r0, r1, c0, c1, bx == by, acc, bad);
}

// One unit per workgroup: block pair and strip from the workgroup number, in the XCD order of sym_unit.
template <int T>
__global__ __launch_bounds__(kSymThreads) void k_sym64_main(int P, int ns, const double4* __restrict__ rec,
                                                            const int32_t* __restrict__ vid,
                                                            const double2* __restrict__ tab,
                                                            const int32_t* __restrict__ meta,
                                                            unsigned long long* __restrict__ acc,
                                                            uint8_t* __restrict__ bad) {
  __shared__ Sym64Lds lds;
  __shared__ double2 ltab[kSymTab];
  const int L = xcd_contiguous(blockIdx.x, gridDim.x);
  int bx, by;
  sym_unit_blocks((P + kSymThreads * T - 1) / (kSymThreads * T), L / ns, bx, by);
  for (int e = threadIdx.x; e < kSymTab; e += kSymThreads) ltab[e] = tab[e];
  sym64_run<T>(lds, P, rec, vid, ltab, meta[1], 0, P, bx, by, ns, L % ns, acc, bad);
}

__device__ __forceinline__ double sym64_value(const unsigned long long* __restrict__ acc,
                                              const uint8_t* __restrict__ bad, int64_t n, int64_t e, double scale, int S,
                                              bool all_bad) {
  const double hi = (double)(long long)acc[e];
  const double lo = (double)(long long)acc[n + e];
  return all_bad || bad[e] ? NAN : ldexp(fma(lo, ldexp(1.0, -kLoBits), hi) * scale, -S);
}

__global__ __launch_bounds__(256) void k_sym64_finish(const unsigned long long* __restrict__ acc,
                                                      const uint8_t* __restrict__ bad,
                                                      const int32_t* __restrict__ meta, int P, double scale,
                                                      double* __restrict__ out) {
  const int S = meta[1];
  const bool all_bad = meta[3] != 0;
  const int64_t n = 2 * (int64_t)P;
  for (int64_t e = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; e < n; e += (int64_t)gridDim.x * blockDim.x)
    out[e] = sym64_value(acc, bad, n, e, scale, S, all_bad);
}

// ------------------------------------------------------------------ batched symmetric form
// Many independent suspensions in one persistent launch.  Each suspension's cycles are contiguous (its
// vesicles in order), its blocks of CB cycles never reach into another suspension, and its units are the
// circulant pairs of its own blocks, so no pair across suspensions is formed.  The units of all
// suspensions are numbered suspension by suspension (row block by row block inside each), and that
// numbering is cut into eight contiguous ranges, one queue per XCD: a workgroup takes units from its own
// XCD's queue by an atomic counter and, once that queue is empty, from the next XCDs' in turn.
// Every unit does the same work (up to the last block of a suspension), so the order needs no sorting.

// Slots of the plan values in the symmetric region's meta array.
constexpr int kMetaUnits = 2;    // total number of units
constexpr int kMetaQueue = 4;    // [kXcds + 1] first unit of each XCD's queue
static_assert(kMetaQueue + kXcds + 1 <= 64, "plan values fit the 256-byte meta slot");
// The queues' counters lie kCountStride ints (a cache line) apart: additions to one line are performed one at a
// time, wherever they come from.
constexpr int kCountStride = kQueueCounters / kXcds;

__device__ __forceinline__ int wave_scan_incl(int x, int lane) {
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const int y = __shfl_up(x, o, 64);
    if (lane >= o) x += y;
  }
  return x;
}

// The range holding x: start[s] <= x < start[s + 1] for one of the n ranges (the last one beyond the end).
__device__ __forceinline__ int range_of(const int32_t* __restrict__ start, int n, int x) {
  int lo = 0, hi = n;
  while (hi - lo > 1) {
    const int mid = (lo + hi) >> 1;
    if (start[mid] <= x)
      lo = mid;
    else
      hi = mid;
  }
  return lo;
}

// Thread 0 takes the next unit from the XCD queues (own XCD's first, then the others' in turn); -1 when all are
// empty.  A queue is looked at before it is added to: without that every workgroup ended with eight additions
// to exhausted queues, 8192 in one line, about 90 us of a call.  Every turn of the loop returns or advances
// `probe`, so it ends.
__device__ __forceinline__ int next_unit(const int32_t* __restrict__ meta, int32_t* __restrict__ count, int xcd,
                                         int& probe) {
  while (probe < kXcds) {
    const int q = xcd + probe < kXcds ? xcd + probe : xcd + probe - kXcds;
    const int lo = meta[kMetaQueue + q], n = meta[kMetaQueue + q + 1] - lo;
    int32_t* c = count + q * kCountStride;
    if (__hip_atomic_load(c, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) < n) {
      const int k = atomicAdd(c, 1);
      if (k < n) return lo + k;
    }
    ++probe;
  }
  return -1;
}

// Disjoint, non-decreasing ranges [max(a_s, every earlier b), max(b_s, that)) of s = 0 .. n - 1 from the ends
// get(s) = (a_s, b_s), by a running maximum; put(s, range) stores them.  Called by 1024 threads, s_w in LDS.
template <class Get, class Put>
__device__ __forceinline__ void disjoint_ranges(int n, int* s_w, Get get, Put put) {
  const int t = threadIdx.x, lane = t & 63, wv = t >> 6;
  int pm = 0;
  for (int base = 0; base < n; base += 1024) {
    const int s = base + t;
    const int2 r = s < n ? get(s) : make_int2(0, 0);
    int x = r.y;  // inclusive running maximum of the ends within the wavefront
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
      const int y = __shfl_up(x, o, 64);
      if (lane >= o) x = max(x, y);
    }
    if (lane == 63) s_w[wv] = x;
    __syncthreads();
    int pre = pm, tot = pm;
    for (int k = 0; k < 16; ++k) {
      pre = k < wv ? max(pre, s_w[k]) : pre;
      tot = max(tot, s_w[k]);
    }
    int ex = __shfl_up(x, 1, 64);  // the maximum over the earlier lanes of this wavefront
    ex = lane == 0 ? pre : max(pre, ex);
    if (s < n) {
      const int v0 = max(r.x, ex);
      put(s, make_int2(v0, max(r.y, v0)));
    }
    pm = tot;
    __syncthreads();
  }
}

// Plan: per suspension s, stab[s] = (first cycle, end cycle, blocks, fixed-point exponent), ustart[s] its
// first unit, pstart[s] its first point (ustart[S], pstart[S]: totals); the cycle table; meta[0] the
// number of cycles, the XCD queues and their zeroed counters.  One workgroup of 1024 threads, in a fixed
// order; the exponent of a suspension is the one the single-suspension plan gives it.
// The suspensions' vesicle ranges are first clamped to [0, M] and made disjoint and non-decreasing
// (vr[s] = (v0, v1), v0 = max(offset s, every earlier end), v1 = max(offset s + 1, v0)): valid offsets are
// unchanged, and no input can make the cycles outrun their table.
__global__ __launch_bounds__(1024) void k_symb_plan(const int2* __restrict__ vrange, const double2* __restrict__ vaux,
                                                    const int32_t* __restrict__ sus_off, int M, int P, int nsus,
                                                    int cb, int ncyc_max, int4* __restrict__ cyc,
                                                    int4* __restrict__ stab, int32_t* __restrict__ ustart,
                                                    int32_t* __restrict__ pstart, int2* __restrict__ vr,
                                                    int32_t* __restrict__ meta, int32_t* __restrict__ count) {
  __shared__ int s_wc[16], s_wu[16];
  const int t = threadIdx.x, lane = t & 63, wv = t >> 6;
  disjoint_ranges(
      nsus, s_wc,
      [&](int s) { return make_int2(min(max(sus_off[s], 0), M), min(max(sus_off[s + 1], 0), M)); },
      [&](int s, int2 r) { vr[s] = r; });
  __syncthreads();
  // cycles and the bound of the partial sums of each suspension, one wavefront per suspension
  for (int s = wv; s < nsus; s += 16) {
    const int2 rs = vr[s];
    const int v0 = rs.x, v1 = rs.y;
    int cnt = 0;
    double fs = 0.0;
    for (int v = v0 + lane; v < v1; v += 64) {
      const int2 r = vrange[v];
      cnt += (max(0, r.y - r.x) + kRing - 1) / kRing;
      fs += vaux[v].x;
    }
#pragma unroll
    for (int m = 32; m >= 1; m >>= 1) cnt += __shfl_xor(cnt, m, 64);
    fs = wave_sum_d(fs);
    if (lane == 0) stab[s] = make_int4(cnt, 0, (cnt + cb - 1) / cb, sym_exponent(fs));
  }
  __syncthreads();
  // exclusive scans over the suspensions: first cycle and first unit
  int runc = 0, runu = 0;
  for (int base = 0; base < nsus; base += 1024) {
    const int s = base + t;
    const int4 st = s < nsus ? stab[s] : make_int4(0, 0, 0, 0);
    const int nu = (int)((int64_t)st.z * (st.z + 1) / 2);
    const int xc = wave_scan_incl(st.x, lane), xu = wave_scan_incl(nu, lane);
    if (lane == 63) {
      s_wc[wv] = xc;
      s_wu[wv] = xu;
    }
    __syncthreads();
    int prec_ = 0, preu = 0, totc = 0, totu = 0;
    for (int k = 0; k < 16; ++k) {
      prec_ += k < wv ? s_wc[k] : 0;
      preu += k < wv ? s_wu[k] : 0;
      totc += s_wc[k];
      totu += s_wu[k];
    }
    if (s < nsus) {
      const int c0 = runc + prec_ + xc - st.x;
      stab[s] = make_int4(c0, c0 + st.x, st.z, st.w);
      ustart[s] = runu + preu + xu - nu;
      const int v0 = vr[s].x;
      pstart[s] = v0 < M ? vrange[v0].x : P;
    }
    runc += totc;
    runu += totu;
    __syncthreads();
  }
  if (t == 0) {
    ustart[nsus] = runu;
    pstart[nsus] = P;
    meta[0] = min(runc, ncyc_max);
    meta[kMetaUnits] = runu;
    const int q = runu / kXcds, r = runu % kXcds;
    for (int x = 0; x <= kXcds; ++x) meta[kMetaQueue + x] = x * q + min(x, r);
  }
  if (t < kXcds) count[t * kCountStride] = 0;
  __syncthreads();
  // the cycles of every vesicle, one wavefront per suspension
  for (int s = wv; s < nsus; s += 16) {
    const int2 rs = vr[s];
    const int v0 = rs.x, v1 = rs.y;
    int c = stab[s].x;
    for (int vb = v0; vb < v1; vb += 64) {
      const int v = vb + lane;
      const int2 r = v < v1 ? vrange[v] : make_int2(0, 0);
      const int n = max(0, r.y - r.x);
      const int cnt = (n + kRing - 1) / kRing;
      const int x = wave_scan_incl(cnt, lane);
      const int first = c + x - cnt;
      for (int k = 0; k < cnt; ++k)
        if (first + k < ncyc_max) cyc[first + k] = make_int4(r.x + kRing * k, min(kRing, n - kRing * k), v, 0);
      c += __shfl(x, 63, 64);
    }
  }
}

// Persistent batched kernel: units from the XCD queues until all are empty (see above).
template <int T>
__global__ __launch_bounds__(kSymThreads) __attribute__((amdgpu_waves_per_eu(T == 2 ? 5 : T == 3 ? 4 : 1))) void k_symb_main(
    int P, const double4* __restrict__ vtab, const double2* __restrict__ vaux, const float4* __restrict__ rec,
    const int4* __restrict__ cyc, const double2* __restrict__ fcyc, const int4* __restrict__ stab,
    const int32_t* __restrict__ ustart, int nsus, const int32_t* __restrict__ meta, int32_t* __restrict__ count,
    unsigned long long* __restrict__ acc) {
  constexpr int CB = kRows * T;
  __shared__ int s_job[2];
  const int xcd = blockIdx.x % kXcds;
  int probe = 0;                    // thread 0: queues found empty so far
  int slo = 0, shi = 0, scur = 0;   // thread 0: unit range of the last suspension found
  for (;;) {
    if (threadIdx.x == 0) {
      const int u = next_unit(meta, count, xcd, probe);
      if (u >= 0 && (u < slo || u >= shi)) {
        scur = range_of(ustart, nsus, u);
        slo = ustart[scur];
        shi = ustart[scur + 1];
      }
      s_job[0] = u;
      s_job[1] = scur;
    }
    __syncthreads();
    const int u = s_job[0], sus = s_job[1];
    __syncthreads();
    if (u < 0) return;
    const int4 st = stab[sus];
    int bx, by;
    sym_unit_blocks(st.z, u - ustart[sus], bx, by);
    const int tc0 = st.x + bx * CB, sc0 = st.x + by * CB;
    sym_eval_unit<T>(P, vtab, vaux, rec, cyc, fcyc, st.w, tc0, min(st.y, tc0 + CB), sc0, min(st.y, sc0 + CB),
                     bx == by, acc);
    __syncthreads();
  }
}

// out = acc 2^-S_s / (4 pi mu_s) for the points of suspension s.
__global__ __launch_bounds__(256) void k_symb_finish(const unsigned long long* __restrict__ acc,
                                                     const int4* __restrict__ stab, const int32_t* __restrict__ pstart,
                                                     const double* __restrict__ mu, int nsus, int P,
                                                     double* __restrict__ out) {
  for (int64_t e = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; e < 2 * (int64_t)P;
       e += (int64_t)gridDim.x * blockDim.x) {
    const int j = (int)(e < P ? e : e - P);
    const int lo = range_of(pstart, nsus, j);
    const double scale = 1.0 / (4.0 * kPi * mu[lo]);
    out[e] = ldexp((double)(long long)acc[e] * scale, -stab[lo].w);
  }
}

// ---- batched float64 form: the float64 symmetric units of many suspensions in one persistent launch, queued
// as above.  Blocks and cycles are cut from each suspension's contiguous points, so the plan holds only point
// ranges, exponents and first units.

// Plan: per suspension stab[s] = (first point, end point, 1 when its bound is not finite, exponent) and its first
// unit (ns strips per block pair of bp points); ranges of vesicles and of points are made disjoint, so no input
// can make the units outrun the host's bound.  One workgroup of 1024 threads, in a fixed order; the others start the
// call.
__global__ __launch_bounds__(1024) void k_symb64_plan(const int2* __restrict__ vrange,
                                                      const double2* __restrict__ vaux,
                                                      const double4* __restrict__ rec,
                                                      const int32_t* __restrict__ sus_off, int M, int P, int nsus,
                                                      int bp, int ns, int4* __restrict__ stab,
                                                      int32_t* __restrict__ ustart, int32_t* __restrict__ pstart,
                                                      int2* __restrict__ vr, int32_t* __restrict__ meta,
                                                      int32_t* __restrict__ count, Sym64Start start) {
  __shared__ int s_w[16];
  if (blockIdx.x > 0) {
    sym64_start(start, blockIdx.x - 1, gridDim.x - 1);
    return;
  }
  const int t = threadIdx.x, lane = t & 63, wv = t >> 6;
  disjoint_ranges(
      nsus, s_w,
      [&](int s) { return make_int2(min(max(sus_off[s], 0), M), min(max(sus_off[s + 1], 0), M)); },
      [&](int s, int2 r) { vr[s] = r; });
  __syncthreads();
  // a wavefront per suspension, or eight lanes where they hold 16 vesicles or fewer on average (1000 suspensions of four:
  // the kernel 70 -> 16 us)
  const int lanes = M > 16 * (int64_t)nsus ? 64 : 8;
  for (int s = t / lanes; s < nsus; s += 1024 / lanes) {
    const int2 rs = vr[s];
    double fs = 0.0;
    for (int v = rs.x + t % lanes; v < rs.y; v += lanes) fs += bound_share(vaux[v].x, vrange[v], rec);
    for (int m = lanes / 2; m >= 1; m >>= 1) fs += __shfl_xor(fs, m, 64);
    if (t % lanes == 0) stab[s] = make_int4(0, 0, isfinite(fs) ? 0 : 1, sym64_exponent(fs));
  }
  __syncthreads();
  disjoint_ranges(
      nsus, s_w,
      [&](int s) {
        const int2 rs = vr[s];
        return rs.x < rs.y ? make_int2(vrange[rs.x].x, vrange[rs.y - 1].y) : make_int2(0, 0);
      },
      [&](int s, int2 r) {
        stab[s].x = r.x;
        stab[s].y = r.y;
        pstart[s] = r.x;
      });
  __syncthreads();
  int run = 0;
  for (int base = 0; base < nsus; base += 1024) {
    const int s = base + t;
    int nu = 0;
    if (s < nsus) {
      const int64_t nb = (stab[s].y - stab[s].x + bp - 1) / bp;
      nu = (int)(nb * (nb + 1) / 2 * ns);
    }
    const int x = wave_scan_incl(nu, lane);
    if (lane == 63) s_w[wv] = x;
    __syncthreads();
    int pre = run, tot = run;
    for (int k = 0; k < 16; ++k) {
      pre += k < wv ? s_w[k] : 0;
      tot += s_w[k];
    }
    if (s < nsus) ustart[s] = pre + x - nu;
    run = tot;
    __syncthreads();
  }
  if (t == 0) {
    ustart[nsus] = run;
    pstart[nsus] = P;
    meta[kMetaUnits] = run;
    const int q = run / kXcds, r = run % kXcds;
    for (int x = 0; x <= kXcds; ++x) meta[kMetaQueue + x] = x * q + min(x, r);
  }
  if (t < kXcds) count[t * kCountStride] = 0;
}

template <int T>
__global__ __launch_bounds__(kSymThreads) void k_symb64_main(int P, int ns, const double4* __restrict__ rec,
                                                             const int32_t* __restrict__ vid,
                                                             const double2* __restrict__ tab,
                                                             const int4* __restrict__ stab,
                                                             const int32_t* __restrict__ ustart, int nsus,
                                                             const int32_t* __restrict__ meta,
                                                             int32_t* __restrict__ count,
                                                             unsigned long long* __restrict__ acc,
                                                             uint8_t* __restrict__ bad) {
  __shared__ Sym64Lds lds;
  __shared__ double2 ltab[kSymTab];
  __shared__ int s_job[2];
  constexpr int BP = kSymThreads * T;
  for (int e = threadIdx.x; e < kSymTab; e += kSymThreads) ltab[e] = tab[e];
  const int xcd = blockIdx.x % kXcds;
  int probe = 0, slo = 0, shi = 0, scur = 0;  // thread 0: queues found empty, units of the last suspension found
  for (;;) {
    if (threadIdx.x == 0) {
      const int u = next_unit(meta, count, xcd, probe);
      if (u >= 0 && (u < slo || u >= shi)) {
        scur = range_of(ustart, nsus, u);
        slo = ustart[scur];
        shi = ustart[scur + 1];
      }
      s_job[0] = u;
      s_job[1] = scur;
    }
    __syncthreads();
    const int u = s_job[0], sus = s_job[1];
    __syncthreads();
    if (u < 0) return;
    const int4 st = stab[sus];
    const int L = u - ustart[sus];
    int bx, by;
    sym_unit_blocks((st.y - st.x + BP - 1) / BP, L / ns, bx, by);
    sym64_run<T>(lds, P, rec, vid, ltab, st.w, st.x, st.y, bx, by, ns, L % ns, acc, bad);
    __syncthreads();
  }
}

__global__ __launch_bounds__(256) void k_symb64_finish(const unsigned long long* __restrict__ acc,
                                                       const uint8_t* __restrict__ bad,
                                                       const int4* __restrict__ stab,
                                                       const int32_t* __restrict__ pstart,
                                                       const double* __restrict__ mu, int nsus, int P,
                                                       double* __restrict__ out) {
  const int64_t n = 2 * (int64_t)P;
  for (int64_t e = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; e < n; e += (int64_t)gridDim.x * blockDim.x) {
    const int s = range_of(pstart, nsus, (int)(e < P ? e : e - P));
    const int4 st = stab[s];
    out[e] = sym64_value(acc, bad, n, e, 1.0 / (4.0 * kPi * mu[s]), st.w, st.z != 0);
  }
}

// Adjoint of the symmetric form, for targets = sources = X (the positions differentiated in both
// roles, w and f held fixed).  With c = 1/(4 pi mu), g = dL/du and phi(r; a, b) = a^T G(r) b:
//   v_k      = sum_{m not in ves(k)} G(X_k - X_m) g_m                (then dL/df = c w v, dL/dw = c f . v)
//   dL/dX_k  = c sum_{m not in ves(k)} H(X_k - X_m),  H(r) = grad phi(r; g_k, F_m) + grad phi(r; F_k, g_m),
//   grad phi(r; a, b) = [ -(a . b) r + a (r . b) + b (a . r) ] / |r|^2 - 2 (a . r)(r . b) r / |r|^4.
// G is even and grad phi odd in r (and symmetric in a, b), so the pair (k, m) adds H to k and -H to m,
// and G(r) g_k to v_m: one evaluation of r, |r|^2, its logarithm and reciprocal serves all four.
// The ring, units and compensation are those of k_sym_main, with g in place of F for v; H is of degree
// -1 in r, so on the rescaled r' = 2^-k r it is computed as H' = 2^k H and scaled back by 2^-k (rows at
// the flush, columns per pair inside the column sum).  Sums are added with float64 atomics.
template <int T>
__global__ __launch_bounds__(kSymThreads) void k_sym_bwd(
    const double4* __restrict__ vtab, const double2* __restrict__ vaux, const float4* __restrict__ recF,
    const float4* __restrict__ recG, const int4* __restrict__ cyc, const double2* __restrict__ gcyc,
    const int32_t* __restrict__ meta, int P, int strips, double* __restrict__ gsum, double* __restrict__ vsum) {
  constexpr int CB = kRows * T;
  __shared__ float4 s_tx[CB][kRing];               // target records (local coordinates, w f)
  __shared__ float2 s_tg[CB][kRing];               // target g
  __shared__ double4 s_tc[CB];                     // (c_A, G_cycle) of each target cycle
  __shared__ double s_tr[CB];                      // R_A^2
  __shared__ int4 s_ti[CB];                        // (vesicle or -1, count, first point, 0)
  __shared__ float4 s_rec[2][kChunk][2 * kRing];   // source cycles (local coordinates, w f), twice
  __shared__ float2 s_reg[2][kChunk][2 * kRing];   // source g, twice
  __shared__ float s_col[2][kSymWaves][kChunk][4][kRing];
  __shared__ double2 s_E[2][kSymWaves][kChunk];

  const int ncyc = meta[0];
  const int nb = meta[2];
  if (nb <= 0) return;
  int bx, by, sc0, sc1;
  if (!sym_unit(nb, strips, CB, ncyc, cyc, bx, by, sc0, sc1)) return;
  const bool diag = bx == by;

  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6, p = lane & 15;
  const int row = tid >> 4;
  const int tc0 = bx * CB, tc1 = min(ncyc, tc0 + CB);

  for (int e = tid; e < CB * kRing; e += kSymThreads) {
    const int t = e / kRing, m = e % kRing;
    const int c = tc0 + t;
    float4 r = make_float4(0.f, 0.f, 0.f, 0.f);
    float2 g = make_float2(0.f, 0.f);
    if (c < tc1) {
      const int4 cy = cyc[c];
      if (m < cy.y) {
        r = recF[cy.x + m];
        const float4 rg = recG[cy.x + m];
        g = make_float2(rg.z, rg.w);
      }
    }
    s_tx[t][m] = r;
    s_tg[t][m] = g;
  }
  for (int t = tid; t < CB; t += kSymThreads) {
    const int c = tc0 + t;
    if (c < tc1) {
      const int4 cy = cyc[c];
      const double4 vt = vtab[cy.z];
      const double2 G = gcyc[c];
      s_tc[t] = make_double4(vt.x, vt.y, G.x, G.y);
      s_tr[t] = vaux[cy.z].y;
      s_ti[t] = make_int4(cy.z, cy.y, cy.x, 0);
    } else {
      s_tc[t] = make_double4(0.0, 0.0, 0.0, 0.0);
      s_tr[t] = 0.0;
      s_ti[t] = make_int4(-1, 0, 0, 0);
    }
  }

  // per target slot k: rescaled position d and -2^-k, the target's F and g (zero when inactive),
  // -1/2 ln2 g, -2^-k for the column gradient, float32 partials of the segment, float64 sums
  float dx[T], dy[T], ns[T], fix[T], fiy[T], gix[T], giy[T], ghx[T], ghy[T];
  float lvx[T], lvy[T], rvx[T], rvy[T], gax[T], gay[T];
  double avx[T], avy[T], agx[T], agy[T];
  int kq[T];
  int actm = 0;
  double Ex = 0.0, Ey = 0.0, Gsx = 0.0, Gsy = 0.0;
#pragma unroll
  for (int k = 0; k < T; ++k) {
    dx[k] = dy[k] = ns[k] = fix[k] = fiy[k] = gix[k] = giy[k] = ghx[k] = ghy[k] = 0.f;
    lvx[k] = lvy[k] = rvx[k] = rvy[k] = gax[k] = gay[k] = 0.f;
    avx[k] = avy[k] = agx[k] = agy[k] = 0.0;
    kq[k] = 0;
  }

  auto setup = [&](int B) {
    const double4 vb = vtab[B];
    const double rb2 = vaux[B].y;
    double ex = 0.0, ey = 0.0;
    actm = 0;
#pragma unroll
    for (int k = 0; k < T; ++k) {
      const int t = k * kRows + row;
      const int4 ti = s_ti[t];
      const double4 tc = s_tc[t];
      const float4 tx = s_tx[t][p];
      const float2 tg = s_tg[t][p];
      const double Dx = tc.x - vb.x, Dy = tc.y - vb.y;
      const double D = fma(Dy, Dy, fma(Dx, Dx, s_tr[t] + rb2));
      int e;
      frexp(D, &e);
      const int kk = min(kMaxShift, max(-kMaxShift, e >> 1));
      const bool rowact = ti.x >= 0 && ti.x != B && (!diag || ti.x < B);
      const bool act = rowact && p < ti.y;
      actm |= act ? (1 << k) : 0;
      const float sc = ldexpf(1.0f, -kk);
      dx[k] = act ? fmaf(tx.x, sc, (float)ldexp(Dx, -kk)) : kFar;
      dy[k] = act ? fmaf(tx.y, sc, (float)ldexp(Dy, -kk)) : 0.f;
      ns[k] = -sc;
      fix[k] = act ? tx.z : 0.f;
      fiy[k] = act ? tx.w : 0.f;
      gix[k] = act ? tg.x : 0.f;
      giy[k] = act ? tg.y : 0.f;
      ghx[k] = kHalfLn2f * gix[k];
      ghy[k] = kHalfLn2f * giy[k];
      kq[k] = kk;
      lvx[k] = lvy[k] = rvx[k] = rvy[k] = gax[k] = gay[k] = 0.f;
      ex += rowact ? (double)kk * tc.z : 0.0;
      ey += rowact ? (double)kk * tc.w : 0.0;
    }
    ex += __shfl_xor(ex, 16, 64);
    ey += __shfl_xor(ey, 16, 64);
    ex += __shfl_xor(ex, 32, 64);
    ey += __shfl_xor(ey, 32, 64);
    Ex = -kLn2d * ex;
    Ey = -kLn2d * ey;
    Gsx = Gsy = 0.0;
  };

  auto flush = [&]() {
#pragma unroll
    for (int k = 0; k < T; ++k) {
      const bool act = (actm >> k) & 1;
      const float pvx = fmaf(kHalfLn2f, lvx[k], rvx[k]);
      const float pvy = fmaf(kHalfLn2f, lvy[k], rvy[k]);
      const double c = -kLn2d * (double)kq[k];
      const double sg = ldexp(1.0, -kq[k]);
      avx[k] += act ? fma(c, Gsx, (double)pvx) : 0.0;
      avy[k] += act ? fma(c, Gsy, (double)pvy) : 0.0;
      agx[k] += act ? sg * (double)gax[k] : 0.0;
      agy[k] += act ? sg * (double)gay[k] : 0.0;
    }
  };

  auto ring = [&](int buf, int cc) {
    const float4* rb = &s_rec[buf][cc][p];
    const float2* gb = &s_reg[buf][cc][p];
    float cvx = 0.f, cvy = 0.f, cgx = 0.f, cgy = 0.f;
#pragma unroll 1
    for (int s = 0; s < kRing; ++s) {
      const float4 sr = rb[s];
      const float2 sg = gb[s];
      float lvcx = 0.f, lvcy = 0.f, lgcx = 0.f, lgcy = 0.f;
#pragma unroll
      for (int k = 0; k < T; ++k) {
        const float rx = fmaf(sr.x, ns[k], dx[k]);
        const float ry = fmaf(sr.y, ns[k], dy[k]);
        const float q = fmaf(ry, ry, rx * rx);
        const float L = __builtin_amdgcn_logf(q);
        const float rho = __builtin_amdgcn_rcpf(q);
        const float ux = rx * rho, uy = ry * rho;
        const float p3 = fmaf(uy, sg.y, ux * sg.x);        // (r . g_j)/q
        const float p2 = fmaf(uy, giy[k], ux * gix[k]);    // (r . g_i)/q
        const float p1 = fmaf(uy, sr.w, ux * sr.z);        // (r . F_j)/q
        const float p4 = fmaf(uy, fiy[k], ux * fix[k]);    // (r . F_i)/q
        // v: G(r) g_j into the row, G(r) g_i into the column
        lvx[k] = fmaf(L, sg.x, lvx[k]);
        lvy[k] = fmaf(L, sg.y, lvy[k]);
        rvx[k] = fmaf(p3, rx, rvx[k]);
        rvy[k] = fmaf(p3, ry, rvy[k]);
        // H' = -(rho (g_i . F_j + F_i . g_j) + 2 (p1 p2 + p3 p4)) r + g_i p1 + F_j p2 + F_i p3 + g_j p4
        const float ab = fmaf(gix[k], sr.z, fmaf(giy[k], sr.w, fmaf(fix[k], sg.x, fiy[k] * sg.y)));
        const float m = fmaf(2.0f, fmaf(p1, p2, p3 * p4), rho * ab);
        const float hx = fmaf(sg.x, p4, fmaf(fix[k], p3, fmaf(sr.z, p2, fmaf(gix[k], p1, -m * rx))));
        const float hy = fmaf(sg.y, p4, fmaf(fiy[k], p3, fmaf(sr.w, p2, fmaf(giy[k], p1, -m * ry))));
        gax[k] += hx;
        gay[k] += hy;
        if (k == 0) {
          lvcx = L * ghx[k];
          lvcy = L * ghy[k];
          lgcx = ns[k] * hx;
          lgcy = ns[k] * hy;
        } else {
          lvcx = fmaf(L, ghx[k], lvcx);
          lvcy = fmaf(L, ghy[k], lvcy);
          lgcx = fmaf(ns[k], hx, lgcx);
          lgcy = fmaf(ns[k], hy, lgcy);
        }
        lvcx = fmaf(p2, rx, lvcx);
        lvcy = fmaf(p2, ry, lvcy);
      }
      cvx = ring_next(cvx) + lvcx;
      cvy = ring_next(cvy) + lvcy;
      cgx = ring_next(cgx) + lgcx;
      cgy = ring_next(cgy) + lgcy;
    }
    // add the four rows: v in the first swap, the gradient in the second
    const auto hv = __builtin_amdgcn_permlane32_swap(bitsu(cvx), bitsu(cvy), false, false);
    const float zv = bitsf(hv[0]) + bitsf(hv[1]);
    const auto rv16 = __builtin_amdgcn_permlane16_swap(bitsu(zv), bitsu(zv), false, false);
    const float totv = bitsf(rv16[0]) + bitsf(rv16[1]);
    const auto hg = __builtin_amdgcn_permlane32_swap(bitsu(cgx), bitsu(cgy), false, false);
    const float zg = bitsf(hg[0]) + bitsf(hg[1]);
    const auto rg16 = __builtin_amdgcn_permlane16_swap(bitsu(zg), bitsu(zg), false, false);
    const float totg = bitsf(rg16[0]) + bitsf(rg16[1]);
    if ((lane & 16) == 0) {
      const int slot = (p + kRing - 1) & (kRing - 1);
      s_col[buf][wv][cc][lane >> 5][slot] = totv;
      s_col[buf][wv][cc][2 + (lane >> 5)][slot] = totg;
    }
  };

  const int nchunks = (sc1 - sc0 + kChunk - 1) / kChunk;
  const bool stager = tid < kChunk * 2 * kRing;
  const int st_cc = tid >> 5, st_q = tid & 31, st_m = st_q & (kRing - 1);
  auto stage_load = [&](int g, float2& gg) {
    float4 r = make_float4(0.f, 0.f, 0.f, 0.f);
    gg = make_float2(0.f, 0.f);
    const int c = sc0 + g * kChunk + st_cc;
    if (stager && c < sc1) {
      const int4 cy = cyc[c];
      const int j = cy.x + (st_m < cy.y ? st_m : 0);
      r = recF[j];
      const float4 rg = recG[j];
      if (st_m >= cy.y) {
        r.z = r.w = 0.f;
      } else {
        gg = make_float2(rg.z, rg.w);
      }
    }
    return r;
  };
  auto stage_store = [&](int buf, const float4& r, const float2& gg) {
    if (stager) {
      s_rec[buf][st_cc][st_q] = r;
      s_reg[buf][st_cc][st_q] = gg;
    }
  };

  // Column sums of chunk g: v (with its log correction) and the gradient, added over the
  // wavefronts in a fixed order, then one float64 atomic addition per (source, component).
  auto reduce = [&](int g, int buf) {
    for (int e = tid; e < kChunk * 4 * kRing; e += kSymThreads) {
      const int cc = e / (4 * kRing), comp = (e / kRing) & 3, m = e & (kRing - 1);
      const int c = sc0 + g * kChunk + cc;
      if (c >= sc1) continue;
      const int4 cy = cyc[c];
      if (m >= cy.y) continue;
      double s = 0.0;
#pragma unroll
      for (int w2 = 0; w2 < kSymWaves; ++w2) s += (double)s_col[buf][w2][cc][comp][m];
      if (comp < 2) {
#pragma unroll
        for (int w2 = 0; w2 < kSymWaves; ++w2) {
          const double2 E = s_E[buf][w2][cc];
          s += comp ? E.y : E.x;
        }
        atomicAdd(&vsum[(size_t)comp * P + cy.x + m], s);
      } else {
        atomicAdd(&gsum[(size_t)(comp - 2) * P + cy.x + m], s);
      }
    }
  };

  int curB = -1;
  {
    float2 gg;
    const float4 r = stage_load(0, gg);
    stage_store(0, r, gg);
  }
  __syncthreads();
  for (int g = 0; g < nchunks; ++g) {
    const int buf = g & 1;
    float2 ngg;
    const float4 nxt = stage_load(g + 1, ngg);
    if (g > 0) reduce(g - 1, buf ^ 1);
    const int cbase = sc0 + g * kChunk;
    const int ncc = min(kChunk, sc1 - cbase);
    for (int cc = 0; cc < ncc; ++cc) {
      const int4 cy = cyc[cbase + cc];
      if (cy.z != curB) {
        if (curB >= 0) flush();
        setup(cy.z);
        curB = cy.z;
      }
      const double2 Gc = gcyc[cbase + cc];
      Gsx += Gc.x;
      Gsy += Gc.y;
      ring(buf, cc);
      if (lane == 0) s_E[buf][wv][cc] = make_double2(Ex, Ey);
    }
    stage_store(buf ^ 1, nxt, ngg);
    __syncthreads();
  }
  if (nchunks > 0) {
    reduce(nchunks - 1, (nchunks - 1) & 1);
    flush();
  }
#pragma unroll
  for (int k = 0; k < T; ++k) {
    const int4 ti = s_ti[k * kRows + row];
    if (ti.x >= 0 && p < ti.y) {
      const int i = ti.z + p;
      atomicAdd(&vsum[i], avx[k]);
      atomicAdd(&vsum[(size_t)P + i], avy[k]);
      atomicAdd(&gsum[i], agx[k]);
      atomicAdd(&gsum[(size_t)P + i], agy[k]);
    }
  }
}

// ---- float64 adjoint for targets = sources, on the blocks, strips and cycles of the float64 forward (points,
// not vesicles; own-vesicle pairs dropped by selects in the units that hold any).
//
// With t = rx rho, u = ry rho, e = rx t, m = 1 - 2e, G = (A c; c B) as in the forward and
//   a = g_ix F_jx + F_ix g_jx,  b = g_iy F_jy + F_iy g_jy,  d = g_ix F_jy + g_iy F_jx + F_ix g_jy + F_iy g_jx,
// H = grad (a A + b B + d c) = ( t (m (a - b) - 2 b) + u d m,  u (m (a - b) - 2 a) - t d m ):
// 55 instructions per unordered pair with the logarithm and the reciprocal.  The four sums are added with
// float64 atomics, as in k_sym_bwd, but to one of kAdjSets copies of each: with strips a point takes up to a few hundred
// additions, which all round at the size of its whole sum.  (Rows in one chain over a unit and one copy gave forces'
// gradients 2.2 times the rounding error at 2000 x 32, and 1.4 times at 504 x 32; the times are the same.)
constexpr int kChunkA = 2;  // source cycles per LDS chunk: 31 KB with the table, so LDS holds five units

// Records, vesicle ids and table, and the cleared sums of v and H: one wavefront per vesicle (its points, offsets
// clamped), the rest dealt over the grid.
__global__ __launch_bounds__(64) void k_sym64_adj_init(const double* __restrict__ X, const double* __restrict__ f,
                                                       const double* __restrict__ w, const int32_t* __restrict__ off,
                                                       int M, int P, double4* __restrict__ rec,
                                                       int32_t* __restrict__ vid, double2* __restrict__ tab,
                                                       double* __restrict__ vsum, double* __restrict__ gsum,
                                                       double* __restrict__ gmore) {
  const int lane = threadIdx.x;
  for (int v = blockIdx.x; v < M; v += gridDim.x) {
    const int j0 = min(max(off[v], 0), P), j1 = max(j0, min(max(off[v + 1], 0), P));
    for (int j = j0 + lane; j < j1; j += 64) {
      rec[j] = make_double4(X[j], X[P + j], w[j] * f[j], w[j] * f[P + j]);
      vid[j] = v;
    }
  }
  const int64_t stride = (int64_t)gridDim.x * 64, first = blockIdx.x * (int64_t)64 + lane;
  for (int64_t e = first; e < 2 * (int64_t)P; e += stride) gsum[e] = 0.0;
  for (int64_t e = first; e < 2 * kAdjSets * (int64_t)P; e += stride) vsum[e] = 0.0;
  for (int64_t e = first; e < 2 * (kAdjSets - 1) * (int64_t)P; e += stride) gmore[e] = 0.0;
  for (int64_t e = first; e < kSymTab; e += stride) tab[e] = half_log_entry((int)e);
}

struct Adj64Lds {
  double4 rec[2][kChunkA][2 * kRing];
  double2 g[2][kChunkA][2 * kRing];
  int32_t vid[2][kChunkA][2 * kRing];
  double col[2][kSymWaves][kChunkA][4][kRing];
};

// One unit of the adjoint: rows [r0, r1) against columns [c0, c1) (as sym64_eval_unit); g planar [2][P].
template <int T>
__device__ __forceinline__ void adj64_eval_unit(Adj64Lds& lds, int P, const double4* __restrict__ rec,
                                                const double* __restrict__ g, const int32_t* __restrict__ vid,
                                                const double2* __restrict__ ltab, int r0, int r1, int c0, int c1,
                                                bool diag, double* __restrict__ gsum, double* __restrict__ vsum) {
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6, p = lane & 15;
  const int row = tid >> 4;
  const bool masked = diag || !(vid[r1 - 1] < vid[c0] || vid[c1 - 1] < vid[r0]);

  double tx[T], ty[T], fx[T], fy[T], gx[T], gy[T], vx[T], vy[T], hx[T], hy[T];
  // the sums of all columns; v, q (the matrix's off-diagonal terms of v) and h are those of a chunk
  double svx[T], svy[T], shx[T], shy[T], qx[T], qy[T];
  int tv[T];
#pragma unroll
  for (int k = 0; k < T; ++k) {
    const int i = r0 + (k * kRows + row) * kRing + p;
    const bool in = i < r1;
    const double4 t = in ? rec[i] : make_double4(kFar64, 0.0, 0.0, 0.0);
    tv[k] = in ? vid[i] : -1;
    tx[k] = t.x;
    ty[k] = t.y;
    fx[k] = t.z;
    fy[k] = t.w;
    gx[k] = in ? g[i] : 0.0;
    gy[k] = in ? g[(size_t)P + i] : 0.0;
    vx[k] = vy[k] = qx[k] = qy[k] = hx[k] = hy[k] = svx[k] = svy[k] = shx[k] = shy[k] = 0.0;
  }

  auto ring = [&](int buf, int cc, auto mask_tag) __attribute__((always_inline)) {
    constexpr bool kMask = decltype(mask_tag)::value;
    const double4* rb = &lds.rec[buf][cc][p];
    const double2* gb = &lds.g[buf][cc][p];
    const int32_t* vb = &lds.vid[buf][cc][p];
    double cvx = 0.0, cvy = 0.0, chx = 0.0, chy = 0.0;
#pragma unroll 1
    for (int s = 0; s < kRing; ++s) {
      const double4 sr = rb[s];
      const double2 sg = gb[s];
      const int sv = kMask ? vb[s] : 0;
      double lvx = 0.0, lvy = 0.0, lhx = 0.0, lhy = 0.0;
#pragma unroll
      for (int k = 0; k < T; ++k) {
        const double rx = tx[k] - sr.x;
        const double ry = ty[k] - sr.y;
        const double q = fma(ry, ry, rx * rx);
        const double l = neg_half_log<true>(q, ltab);
        const double rho = recip(q);
        const double t = rx * rho, u = ry * rho;
        const double e = rx * t;
        const double A = l + e, B = fma(ry, u, l), c = ry * t, m = fma(-2.0, e, 1.0);
        const double a = fma(fx[k], sg.x, gx[k] * sr.z);
        const double b = fma(fy[k], sg.y, gy[k] * sr.w);
        const double d = fma(gx[k], sr.w, fma(gy[k], sr.z, fma(fx[k], sg.y, fy[k] * sg.x)));
        const double n = m * (a - b), dm = d * m;
        const double Hx = fma(t, fma(-2.0, b, n), u * dm);
        const double Hy = fma(u, fma(-2.0, a, n), -t * dm);
        const double nvx = fma(A, sg.x, vx[k]), nqx = fma(c, sg.y, qx[k]);
        const double nvy = fma(B, sg.y, vy[k]), nqy = fma(c, sg.x, qy[k]);
        const double nhx = hx[k] + Hx, nhy = hy[k] + Hy;
        const double nlvx = fma(A, gx[k], k == 0 ? c * gy[k] : fma(c, gy[k], lvx));
        const double nlvy = fma(c, gx[k], k == 0 ? B * gy[k] : fma(B, gy[k], lvy));
        const double nlhx = k == 0 ? Hx : lhx + Hx, nlhy = k == 0 ? Hy : lhy + Hy;
        const bool act = !kMask || (diag ? tv[k] < sv : tv[k] != sv);
        vx[k] = act ? nvx : vx[k];
        vy[k] = act ? nvy : vy[k];
        qx[k] = act ? nqx : qx[k];
        qy[k] = act ? nqy : qy[k];
        hx[k] = act ? nhx : hx[k];
        hy[k] = act ? nhy : hy[k];
        lvx = act ? nlvx : lvx;
        lvy = act ? nlvy : lvy;
        lhx = act ? nlhx : lhx;
        lhy = act ? nlhy : lhy;
      }
      cvx = ring_next64(cvx) + lvx;
      cvy = ring_next64(cvy) + lvy;
      chx = ring_next64(chx) - lhx;
      chy = ring_next64(chy) - lhy;
    }
    // add the four rows of the wavefront (both halves of each double swapped alike): v, then H
    auto rows4 = [&](double x, double y) {
      const unsigned long long bx = dlo(x), by = dlo(y);
      const auto hl = __builtin_amdgcn_permlane32_swap((unsigned)bx, (unsigned)by, false, false);
      const auto hh = __builtin_amdgcn_permlane32_swap((unsigned)(bx >> 32), (unsigned)(by >> 32), false, false);
      const double z = dfrom(hl[0], hh[0]) + dfrom(hl[1], hh[1]);
      const unsigned long long bz = dlo(z);
      const auto gl = __builtin_amdgcn_permlane16_swap((unsigned)bz, (unsigned)bz, false, false);
      const auto gh = __builtin_amdgcn_permlane16_swap((unsigned)(bz >> 32), (unsigned)(bz >> 32), false, false);
      return dfrom(gl[0], gh[0]) + dfrom(gl[1], gh[1]);
    };
    const double totv = rows4(cvx, cvy);
    const double toth = rows4(chx, chy);
    if ((lane & 16) == 0) {
      const int slot = (p + kRing - 1) & (kRing - 1);
      lds.col[buf][wv][cc][lane >> 5][slot] = totv;
      lds.col[buf][wv][cc][2 + (lane >> 5)][slot] = toth;
    }
  };

  const int ncyc = (c1 - c0 + kRing - 1) / kRing;
  const int nchunks = (ncyc + kChunkA - 1) / kChunkA;
  const bool stager = tid < kChunkA * 2 * kRing;
  const int st_cc = tid >> 5, st_q = tid & 31;
  struct Src {
    double4 r;
    double2 g;
    int v;
  };
  auto stage_load = [&](int ch) {
    Src o = {make_double4(0.0, 0.0, 0.0, 0.0), make_double2(0.0, 0.0), -1};
    const int j = c0 + (ch * kChunkA + st_cc) * kRing + (st_q & (kRing - 1));
    if (stager && ch < nchunks) {
      const int jj = min(j, c1 - 1);  // past the end: the last point with zero force and g
      o.r = rec[jj];
      o.v = vid[jj];
      if (j >= c1)
        o.r.z = o.r.w = 0.0;
      else
        o.g = make_double2(g[jj], g[(size_t)P + jj]);
    }
    return o;
  };
  auto stage_store = [&](int buf, const Src& o) {
    if (stager) {
      lds.rec[buf][st_cc][st_q] = o.r;
      lds.g[buf][st_cc][st_q] = o.g;
      lds.vid[buf][st_cc][st_q] = o.v;
    }
  };
  // column sums of a chunk: v and H added over the wavefronts in a fixed order, one float64 atomic addition per
  // (source, quantity, component)
  auto reduce = [&](int ch, int buf) {
    if (tid >= kChunkA * 4 * kRing) return;
    const int cc = tid >> 6, comp = (tid >> 4) & 3, m = tid & (kRing - 1);
    const int j = c0 + (ch * kChunkA + cc) * kRing + m;
    if (j >= c1) return;
    const double v = ((lds.col[buf][0][cc][comp][m] + lds.col[buf][1][cc][comp][m]) + lds.col[buf][2][cc][comp][m]) +
                     lds.col[buf][3][cc][comp][m];
    double* dst = comp < 2 ? vsum : gsum;
    atomicAdd(&dst[(size_t)(comp & 1) * P + j], v);
  };

  stage_store(0, stage_load(0));
  __syncthreads();
  for (int ch = 0; ch < nchunks; ++ch) {
    const int buf = ch & 1;
    const Src nxt = stage_load(ch + 1);
    if (ch > 0) reduce(ch - 1, buf ^ 1);
    const int ncc = min(kChunkA, ncyc - ch * kChunkA);
    if (masked)
      for (int cc = 0; cc < ncc; ++cc) ring(buf, cc, std::true_type{});
    else
      for (int cc = 0; cc < ncc; ++cc) ring(buf, cc, std::false_type{});
#pragma unroll
    for (int k = 0; k < T; ++k) {
      svx[k] += vx[k] + qx[k];
      svy[k] += vy[k] + qy[k];
      shx[k] += hx[k];
      shy[k] += hy[k];
      vx[k] = vy[k] = qx[k] = qy[k] = hx[k] = hy[k] = 0.0;
    }
    stage_store(buf ^ 1, nxt);
    __syncthreads();
  }
  reduce(nchunks - 1, (nchunks - 1) & 1);
#pragma unroll
  for (int k = 0; k < T; ++k) {
    const int i = r0 + (k * kRows + row) * kRing + p;
    if (i < r1) {
      atomicAdd(&vsum[i], svx[k]);
      atomicAdd(&vsum[(size_t)P + i], svy[k]);
      atomicAdd(&gsum[i], shx[k]);
      atomicAdd(&gsum[(size_t)P + i], shy[k]);
    }
  }
}

// One unit per workgroup, as k_sym64_main.
template <int T>
__global__ __launch_bounds__(kSymThreads) void k_sym64_bwd(int P, int ns, const double4* __restrict__ rec,
                                                           const double* __restrict__ g,
                                                           const int32_t* __restrict__ vid,
                                                           const double2* __restrict__ tab, double* __restrict__ gsum,
                                                           double* __restrict__ gmore, double* __restrict__ vsum) {
  __shared__ Adj64Lds lds;
  __shared__ double2 ltab[kSymTab];
  constexpr int BP = kSymThreads * T;
  const int L = xcd_contiguous(blockIdx.x, gridDim.x);
  int bx, by;
  sym_unit_blocks((P + BP - 1) / BP, L / ns, bx, by);
  const int c0 = by * BP + (L % ns) * (BP / ns), c1 = min(P, c0 + BP / ns);
  if (c0 >= c1) return;
  for (int e = threadIdx.x; e < kSymTab; e += kSymThreads) ltab[e] = tab[e];
  // a row point's additions differ in the strip, a column point's in the row block
  const int set = (bx + L % ns) % kAdjSets;
  if (set > 0) gsum = gmore + (size_t)(set - 1) * 2 * P;
  vsum += (size_t)set * 2 * P;
  // the diagonal block's rows past the strip hold no pair of it; half the rows or fewer take the narrower form
  const int r0 = bx * BP, r1 = min(bx == by ? c1 : P, r0 + BP);
  if (T > 1 && r1 - r0 <= kSymThreads)
    adj64_eval_unit<1>(lds, P, rec, g, vid, ltab, r0, r1, c0, c1, bx == by, gsum, vsum);
  else
    adj64_eval_unit<T>(lds, P, rec, g, vid, ltab, r0, r1, c0, c1, bx == by, gsum, vsum);
}

__global__ __launch_bounds__(256) void k_zero_f64(double* __restrict__ a, int64_t n) {
  for (int64_t e = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; e < n; e += (int64_t)gridDim.x * blockDim.x)
    a[e] = 0.0;
}

__global__ __launch_bounds__(256) void k_add_f64(double* __restrict__ a, const double* __restrict__ b, int64_t n) {
  for (int64_t e = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; e < n; e += (int64_t)gridDim.x * blockDim.x)
    a[e] += b[e];
}

// dL/dX = c gsum (in place), dL/df = c w v, dL/dw = c f . v
__global__ __launch_bounds__(256) void k_sym_bwd_finish(const double* __restrict__ vsum, const double* __restrict__ f,
                                                        const double* __restrict__ w, int P, double scale,
                                                        double* __restrict__ gX, double* __restrict__ gf,
                                                        double* __restrict__ gw) {
  for (int j = blockIdx.x * blockDim.x + threadIdx.x; j < P; j += gridDim.x * blockDim.x) {
    if (gX) {
      gX[j] *= scale;
      gX[P + j] *= scale;
    }
    const double vx = scale * vsum[j], vy = scale * vsum[P + j];
    if (gf) {
      gf[j] = w[j] * vx;
      gf[P + j] = w[j] * vy;
    }
    if (gw) gw[j] = f[j] * vx + f[P + j] * vy;
  }
}

// The same after the float64 adjoint, whose sums come in kAdjSets copies.
__global__ __launch_bounds__(256) void k_sym64_bwd_finish(const double* __restrict__ vsum,
                                                          const double* __restrict__ gmore,
                                                          const double* __restrict__ f, const double* __restrict__ w,
                                                          int P, double scale, double* __restrict__ gX,
                                                          double* __restrict__ gf, double* __restrict__ gw) {
  const size_t n = 2 * (size_t)P;
  for (int j = blockIdx.x * blockDim.x + threadIdx.x; j < P; j += gridDim.x * blockDim.x) {
    double hx = gX[j], hy = gX[P + j], vx = vsum[j], vy = vsum[P + j];
#pragma unroll
    for (int k = 1; k < kAdjSets; ++k) {
      hx += gmore[(k - 1) * n + j];
      hy += gmore[(k - 1) * n + P + j];
      vx += vsum[k * n + j];
      vy += vsum[k * n + P + j];
    }
    gX[j] = hx * scale;
    gX[P + j] = hy * scale;
    vx *= scale;
    vy *= scale;
    if (gf) {
      gf[j] = w[j] * vx;
      gf[P + j] = w[j] * vy;
    }
    if (gw) gw[j] = f[j] * vx + f[P + j] * vy;
  }
}

__global__ __launch_bounds__(256) void k_sym_finish(const unsigned long long* __restrict__ acc,
                                                    const int32_t* __restrict__ meta, int P, double scale,
                                                    double* __restrict__ out) {
  const int S = meta[1];
  for (int64_t e = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; e < 2 * (int64_t)P;
       e += (int64_t)gridDim.x * blockDim.x)
    out[e] = ldexp((double)(long long)acc[e] * scale, -S);
}

}  // namespace

static inline hipStream_t Sx_(void* s) { return reinterpret_cast<hipStream_t>(s); }

int sym_cycles_per_block(int T) { return kRows * T; }

int64_t sym_max_cycles(int P, int M) { return (int64_t)P / kRing + (int64_t)M + 1; }

int64_t sym_max_blocks(int P, int M, int T) {
  const int cb = sym_cycles_per_block(T);
  return (sym_max_cycles(P, M) + cb - 1) / cb;
}

int64_t sym_units(int64_t nb) {
  if (nb <= 0) return 0;
  const int64_t h = nb / 2;
  return (nb & 1) ? nb * (h + 1) : nb * h + h;
}

bool sym_fits(int P, int M, int T) { return sym_units(sym_max_blocks(P, M, T)) <= (int64_t)INT32_MAX; }

// Above this many vesicles the counting of those before (M^2 / 2 offsets) and the units' sums of M bounds would cost
// more than the launches they save.
bool sym_fused(int M) { return M <= kSymFused; }

hipError_t launch_backward_symmetric(int T, int ns, int P, int M, const PreparedView& pvF, const PreparedView& pvG,
                                     const SymmetricView& sv, double* vsum, const SymmetricInput& in,
                                     double scale, double* grad_points, double* grad_f, double* grad_w,
                                     void* stream) {
  if (P == 0) return hipSuccess;
  if (!grad_points || !vsum) return hipErrorInvalidValue;
  const double* f = in.f;
  const double* w = in.w;
  hipStream_t st = Sx_(stream);
  const int cb = sym_cycles_per_block(T);
  const int ncyc_max = (int)sym_max_cycles(P, M);
  const int nb_max = (int)sym_max_blocks(P, M, T);
  if (sym_fused(M)) {
    hipLaunchKernelGGL(k_sym_prepare<true>, dim3(M), dim3(64), 0, st, in.pts, f, w, in.g, in.off, M, P, cb, ncyc_max,
                       pvF, static_cast<float4*>(pvG.rec), sv.cyc, sv.fcyc,
                       sv.meta, reinterpret_cast<unsigned long long*>(grad_points),
                       reinterpret_cast<unsigned long long*>(vsum));
  } else {
    hipError_t e = launch_prepare(P32C, in.pts, f, w, in.off, M, P, pvF, stream);
    if (e == hipSuccess) e = launch_prepare(P32C, in.pts, in.g, nullptr, in.off, M, P, pvG, stream);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_sym_plan, dim3(1), dim3(1024), 0, st, pvF.vrange, pvF.vaux, M, cb, ncyc_max, sv.cyc, sv.meta);
    const int cgrid = (int)std::min<int64_t>((2 * (int64_t)P + 255) / 256, 4096);
    // cycle sums of g (its float64 copy is the f64 array of the g-prepared region)
    hipLaunchKernelGGL(k_sym_cycles, dim3(cgrid), dim3(256), 0, st, sv.cyc, sv.meta, pvG.f64, P, sv.fcyc, sv.acc);
    hipLaunchKernelGGL(k_zero_f64, dim3(cgrid), dim3(256), 0, st, grad_points, 2 * (int64_t)P);
    hipLaunchKernelGGL(k_zero_f64, dim3(cgrid), dim3(256), 0, st, vsum, 2 * (int64_t)P);
  }
  const dim3 grid((unsigned)(sym_units(nb_max) * ns));
  const float4* recF = static_cast<const float4*>(pvF.rec);
  const float4* recG = static_cast<const float4*>(pvG.rec);
  switch (T) {
#define VESNET_SYMB_CASE(TT)                                                                                   \
  case TT:                                                                                                     \
    hipLaunchKernelGGL(k_sym_bwd<TT>, grid, dim3(kSymThreads), 0, st, pvF.vtab, pvF.vaux, recF, recG, sv.cyc,  \
                       sv.fcyc, sv.meta, P, ns, grad_points, vsum);                                             \
    break;
    VESNET_SYMB_CASE(1) VESNET_SYMB_CASE(2) VESNET_SYMB_CASE(3) VESNET_SYMB_CASE(4)
#undef VESNET_SYMB_CASE
    default: return hipErrorInvalidValue;
  }
  const int fgrid = (P + 255) / 256 < 16384 ? (P + 255) / 256 : 16384;
  hipLaunchKernelGGL(k_sym_bwd_finish, dim3(fgrid), dim3(256), 0, st, vsum, f, w, P, scale, grad_points, grad_f,
                     grad_w);
  return hipGetLastError();
}

hipError_t launch_backward_symmetric64(int T, int ns, int P, int M, const double* X, const double* f, const double* w,
                                       const int32_t* off, const double* gout, const Adjoint64View& av, double scale,
                                       double* grad_points, double* grad_f, double* grad_w, void* stream) {
  if (P == 0) return hipSuccess;
  if (!grad_points || ns < 1 || kRows % ns != 0) return hipErrorInvalidValue;
  hipStream_t st = Sx_(stream);
  const int igrid = (int)std::min<int64_t>(std::max<int64_t>(M, (2 * (int64_t)P + 255) / 256), 65535);
  hipLaunchKernelGGL(k_sym64_adj_init, dim3(igrid), dim3(64), 0, st, X, f, w, off, M, P, av.rec, av.vid, av.tab, av.vsum,
                     grad_points, av.gmore);
  const int64_t units = sym_units(sym64_blocks(P, T)) * ns;
  if (units > (int64_t)INT32_MAX) return hipErrorInvalidValue;
  const dim3 grid((unsigned)units);
  switch (T) {
#define VESNET_ADJ64_CASE(TT)                                                                                     \
  case TT:                                                                                                        \
    hipLaunchKernelGGL(k_sym64_bwd<TT>, grid, dim3(kSymThreads), 0, st, P, ns, av.rec, gout, av.vid, av.tab,      \
                       grad_points, av.gmore, av.vsum);                                                           \
    break;
    VESNET_ADJ64_CASE(1) VESNET_ADJ64_CASE(2) VESNET_ADJ64_CASE(3) VESNET_ADJ64_CASE(4)
#undef VESNET_ADJ64_CASE
    default: return hipErrorInvalidValue;
  }
  const int fgrid = (P + 255) / 256 < 16384 ? (P + 255) / 256 : 16384;
  hipLaunchKernelGGL(k_sym64_bwd_finish, dim3(fgrid), dim3(256), 0, st, av.vsum, av.gmore, f, w, P, scale, grad_points,
                     grad_f, grad_w);
  return hipGetLastError();
}

hipError_t launch_add_f64(double* a, const double* b, int64_t n, void* stream) {
  if (n <= 0) return hipSuccess;
  const int grid = (int)std::min<int64_t>((n + 255) / 256, 4096);
  hipLaunchKernelGGL(k_add_f64, dim3(grid), dim3(256), 0, Sx_(stream), a, b, n);
  return hipGetLastError();
}

int64_t symb_max_units(int P, int M, int S, int T) {
  // the blocks of all suspensions number at most (cycles / CB) + S, and n (n + 1) / 2 is superadditive
  return sym_units(sym_max_blocks(P, M, T) + S);
}

// Cached after the first query (every device this library runs on is a gfx950).
int symb_units_per_cu(int T) {
  static std::atomic<int> cache[5] = {};
  if (T < 1 || T > 4) return 1;
  int n = cache[T].load(std::memory_order_relaxed);
  if (n > 0) return n;
  hipError_t e = hipErrorInvalidValue;
  switch (T) {
    case 1: e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&n, k_symb_main<1>, kSymThreads, 0); break;
    case 2: e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&n, k_symb_main<2>, kSymThreads, 0); break;
    case 3: e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&n, k_symb_main<3>, kSymThreads, 0); break;
    default: e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&n, k_symb_main<4>, kSymThreads, 0); break;
  }
  if (e != hipSuccess || n <= 0) return 1;
  cache[T].store(n, std::memory_order_relaxed);
  return n;
}

hipError_t launch_batched_symmetric(int T, int grid, int P, int M, const PreparedView& pv, const SymmetricView& sv,
                                    const SymBatchView& bv, const int32_t* sus_off, const int32_t* off, int S,
                                    const double* mu, double* out, void* stream) {
  if (P == 0 || S == 0) return hipSuccess;
  if (grid < 1) return hipErrorInvalidValue;
  hipStream_t st = Sx_(stream);
  const int cb = sym_cycles_per_block(T);
  const int ncyc_max = (int)sym_max_cycles(P, M);
  hipLaunchKernelGGL(k_symb_plan, dim3(1), dim3(1024), 0, st, pv.vrange, pv.vaux, sus_off, M, P, S, cb, ncyc_max,
                     sv.cyc, bv.stab, bv.ustart, bv.pstart, bv.vr, sv.meta, bv.count);
  const int cgrid = (int)std::min<int64_t>((2 * (int64_t)P + 255) / 256, 4096);
  hipLaunchKernelGGL(k_sym_cycles, dim3(cgrid), dim3(256), 0, st, sv.cyc, sv.meta, pv.f64, P, sv.fcyc, sv.acc);
  const float4* rec = static_cast<const float4*>(pv.rec);
  switch (T) {
#define VESNET_SYMB_MAIN(TT)                                                                                     \
  case TT:                                                                                                       \
    hipLaunchKernelGGL(k_symb_main<TT>, dim3(grid), dim3(kSymThreads), 0, st, P, pv.vtab, pv.vaux, rec, sv.cyc, \
                       sv.fcyc, bv.stab, bv.ustart, S, sv.meta, bv.count, sv.acc);                                \
    break;
    VESNET_SYMB_MAIN(1) VESNET_SYMB_MAIN(2) VESNET_SYMB_MAIN(3) VESNET_SYMB_MAIN(4)
#undef VESNET_SYMB_MAIN
    default: return hipErrorInvalidValue;
  }
  const int64_t n = 2 * (int64_t)P;
  const int fgrid = (int)((n + 255) / 256 < 16384 ? (n + 255) / 256 : 16384);
  hipLaunchKernelGGL(k_symb_finish, dim3(fgrid), dim3(256), 0, st, sv.acc, bv.stab, bv.pstart, mu, S, P, out);
  return hipGetLastError();
}

int64_t sym64_blocks(int64_t P, int T) { return (P + kSymThreads * T - 1) / (kSymThreads * T); }

// Workgroups that start a float64 call.
static int sym64_start_grid(int P) { return (int)std::min<int64_t>((4 * (int64_t)P + 1023) / 1024, 1024); }

static Sym64Start sym64_start_of(const Symmetric64View& sv, int P) {
  return {sv.acc, reinterpret_cast<uint32_t*>(sv.bad), sv.tab, P};
}

int64_t symb64_max_units(int P, int S, int T, int ns) {
  // the blocks of all suspensions number at most P / (256 T) + S, and n (n + 1) / 2 is superadditive
  return sym_units(sym64_blocks(P, T) + S) * ns;
}

// Cached after the first query (every device this library runs on is a gfx950).
int symb64_units_per_cu(int T) {
  static std::atomic<int> cache[3] = {};
  if (T < 1 || T > 2) return 1;
  int n = cache[T].load(std::memory_order_relaxed);
  if (n > 0) return n;
  const hipError_t e = T == 1 ? hipOccupancyMaxActiveBlocksPerMultiprocessor(&n, k_symb64_main<1>, kSymThreads, 0)
                              : hipOccupancyMaxActiveBlocksPerMultiprocessor(&n, k_symb64_main<2>, kSymThreads, 0);
  if (e != hipSuccess || n <= 0) return 1;
  cache[T].store(n, std::memory_order_relaxed);
  return n;
}

hipError_t launch_batched_symmetric64(int T, int ns, int grid, int P, int M, const PreparedView& pv,
                                      const Symmetric64View& sv, const SymBatchView& bv, const int32_t* sus_off, int S,
                                      const double* mu, double* out, void* stream) {
  if (P == 0 || S == 0) return hipSuccess;
  if (grid < 1 || ns < 1 || kRows % ns != 0) return hipErrorInvalidValue;
  hipStream_t st = Sx_(stream);
  const double4* rec = static_cast<const double4*>(pv.rec);
  hipLaunchKernelGGL(k_symb64_plan, dim3(1 + sym64_start_grid(P)), dim3(1024), 0, st, pv.vrange, pv.vaux, rec, sus_off, M,
                     P, S, kSymThreads * T, ns, bv.stab, bv.ustart, bv.pstart, bv.vr, sv.meta, bv.count,
                     sym64_start_of(sv, P));
  if (T == 1)
    hipLaunchKernelGGL(k_symb64_main<1>, dim3(grid), dim3(kSymThreads), 0, st, P, ns, rec, pv.vid, sv.tab, bv.stab,
                       bv.ustart, S, sv.meta, bv.count, sv.acc, sv.bad);
  else if (T == 2)
    hipLaunchKernelGGL(k_symb64_main<2>, dim3(grid), dim3(kSymThreads), 0, st, P, ns, rec, pv.vid, sv.tab, bv.stab,
                       bv.ustart, S, sv.meta, bv.count, sv.acc, sv.bad);
  else
    return hipErrorInvalidValue;
  const int64_t n = 2 * (int64_t)P;
  const int fgrid = (int)((n + 255) / 256 < 16384 ? (n + 255) / 256 : 16384);
  hipLaunchKernelGGL(k_symb64_finish, dim3(fgrid), dim3(256), 0, st, sv.acc, sv.bad, bv.stab, bv.pstart, mu, S, P, out);
  return hipGetLastError();
}

hipError_t launch_forward_symmetric64(int T, int ns, int P, int M, const PreparedView& pv, const Symmetric64View& sv,
                                      double scale, double* out, void* stream) {
  if (P == 0) return hipSuccess;
  if (ns < 1 || kRows % ns != 0) return hipErrorInvalidValue;
  hipStream_t st = Sx_(stream);
  hipLaunchKernelGGL(k_sym64_init, dim3(sym64_start_grid(P)), dim3(1024), 0, st, pv.vaux, pv.vrange,
                     static_cast<const double4*>(pv.rec), M, sym64_start_of(sv, P), sv.meta);
  const int64_t units = sym_units(sym64_blocks(P, T)) * ns;
  if (units > (int64_t)INT32_MAX) return hipErrorInvalidValue;
  const dim3 grid((unsigned)units);
  const double4* rec = static_cast<const double4*>(pv.rec);
  switch (T) {
#define VESNET_SYM64_CASE(TT)                                                                                       \
  case TT:                                                                                                          \
    hipLaunchKernelGGL(k_sym64_main<TT>, grid, dim3(kSymThreads), 0, st, P, ns, rec, pv.vid, sv.tab, sv.meta, sv.acc, \
                       sv.bad);                                                                                     \
    break;
    VESNET_SYM64_CASE(1) VESNET_SYM64_CASE(2) VESNET_SYM64_CASE(3) VESNET_SYM64_CASE(4)
#undef VESNET_SYM64_CASE
    default: return hipErrorInvalidValue;
  }
  const int64_t n = 2 * (int64_t)P;
  const int fgrid = (int)((n + 255) / 256 < 16384 ? (n + 255) / 256 : 16384);
  hipLaunchKernelGGL(k_sym64_finish, dim3(fgrid), dim3(256), 0, st, sv.acc, sv.bad, sv.meta, P, scale, out);
  return hipGetLastError();
}

hipError_t launch_forward_symmetric(int T, int ns, int P, int M, const PreparedView& pv, const SymmetricView& sv,
                                    const SymmetricInput* in, double scale, double* out, void* stream) {
  if (P == 0) return hipSuccess;
  hipStream_t st = Sx_(stream);
  const int cb = sym_cycles_per_block(T);
  const int ncyc_max = (int)sym_max_cycles(P, M);
  const int nb_max = (int)sym_max_blocks(P, M, T);
  // a wavefront per vesicle is a serial chain: with few large vesicles the separate kernels, whose cycle sums and
  // clearing use the whole chip, are faster (4 x 16,384 1.26 ms against 1.29, 16 x 2,048 359 us against 357; the adjoint,
  // which they prepare twice, gains at every size)
  const bool fused = in != nullptr && sym_fused(M) && P <= 2048 * (int64_t)M;
  if (fused) {
    hipLaunchKernelGGL(k_sym_prepare<false>, dim3(M), dim3(64), 0, st, in->pts, in->f, in->w, nullptr, in->off, M, P, cb,
                       ncyc_max, pv, nullptr, sv.cyc, sv.fcyc, sv.meta, sv.acc, nullptr);
  } else {
    if (in != nullptr) {
      const hipError_t e = launch_prepare(P32C, in->pts, in->f, in->w, in->off, M, P, pv, stream);
      if (e != hipSuccess) return e;
    }
    hipLaunchKernelGGL(k_sym_plan, dim3(1), dim3(1024), 0, st, pv.vrange, pv.vaux, M, cb, ncyc_max, sv.cyc, sv.meta);
    const int cgrid = (int)std::min<int64_t>((2 * (int64_t)P + 255) / 256, 4096);
    hipLaunchKernelGGL(k_sym_cycles, dim3(cgrid), dim3(256), 0, st, sv.cyc, sv.meta, pv.f64, P, sv.fcyc, sv.acc);
  }
  const dim3 grid((unsigned)(sym_units(nb_max) * ns));
  const float4* rec = static_cast<const float4*>(pv.rec);
  switch (T) {
#define VESNET_SYM_CASE(TT)                                                                                    \
  case TT:                                                                                                     \
    if (fused)                                                                                                 \
      hipLaunchKernelGGL((k_sym_main<TT, true>), grid, dim3(kSymThreads), 0, st, P, ns, pv.vtab, pv.vaux, rec, \
                         sv.cyc, sv.fcyc, sv.meta, M, sv.acc);                                                 \
    else                                                                                                       \
      hipLaunchKernelGGL((k_sym_main<TT, false>), grid, dim3(kSymThreads), 0, st, P, ns, pv.vtab, pv.vaux,     \
                         rec, sv.cyc, sv.fcyc, sv.meta, M, sv.acc);                                            \
    break;
    VESNET_SYM_CASE(1) VESNET_SYM_CASE(2) VESNET_SYM_CASE(3) VESNET_SYM_CASE(4) VESNET_SYM_CASE(8)
#undef VESNET_SYM_CASE
    default: return hipErrorInvalidValue;
  }
  const int64_t n = 2 * (int64_t)P;
  const int fgrid = (int)((n + 255) / 256 < 16384 ? (n + 255) / 256 : 16384);
  hipLaunchKernelGGL(k_sym_finish, dim3(fgrid), dim3(256), 0, st, sv.acc, sv.meta, P, scale, out);
  return hipGetLastError();
}

}  // namespace vesnet

// The GP's negative log likelihood and its gradient in the hyperparameters,
// evaluated on the device in fp64 (Sec. 4.3: the noise level and the other
// hyperparameters are learned by maximum likelihood).  The search itself (the
// box-constrained L-BFGS of host_mle.cpp) stays on the host and calls this
// once per trial point.
//
// With r = y - c, K = k_theta(X, X) + tau2 I (m x m), K = L L^T, u = L^-1 r and
// W = alpha alpha^T - K^-1:
//   NLL = 1/2 u^T u + 1/2 log det K + m/2 log(2 pi),   alpha = K^-1 r = L^-T u
//   dNLL/dtheta_p = -1/2 sum_ij W_ij (dK/dtheta_p)_ij
// with the derivatives of the covariance written out in host_mle.cpp.
//
// Matrices are 16 x 16 blocks, m padded to a multiple of 16 with identity rows
// (their covariance with real rows is 0, their diagonal 1, their r 0: log det,
// the quadratic form and the gradient do not see them).  The kernels of one
// evaluation, on one stream:
//   W. (warp learned) the warped inputs and their derivatives;
//   K. K, one 16 x 16 block per workgroup;
//   A. one workgroup (8 waves): the Cholesky factor L by 16-column block
//      steps: the diagonal block factored and inverted by one wave in
//      registers (a rank-4 update per four columns on v_mfma_f64_16x16x4f64), the
//      panel below it as the product with that inverse and the trailing
//      update, both on the matrix cores, and u = L^-1 r by forward
//      substitution alongside; the next diagonal block is factored as soon
//      as it is updated, by a wave whose SIMD the others leave free;
// and, when the gradient is wanted,
//   T. L^-1 and alpha = L^-T u, one block column per workgroup (the columns
//      are independent);
//   B. the gradient, one lower block per workgroup: the block of
//      K^-1 = L^-T L^-1 on the matrix cores, then one element of W per
//      thread, the covariance and its derivatives recomputed, partial sums
//      per workgroup.
// The kernels write their results (status, pivot products, |u|^2 per block,
// partial gradient sums) straight into pinned host memory, and the host adds
// them.  Every operation is in double and every sum has a fixed order, so an
// evaluation is deterministic.
#include <hip/hip_runtime.h>

#include <cmath>
#include <cstring>
#include <utility>
#include <vector>

#include "internal.h"

namespace scoot {
namespace {

typedef double d2_t __attribute__((ext_vector_type(2)));
typedef double d4_t __attribute__((ext_vector_type(4)));

constexpr int kNllWaves = 8;
constexpr int kNllThreads = kNllWaves * 64;
constexpr int kMaxTheta = 3 * SCOOT_MAX_DIM + 2;
constexpr int kGradThreads = 256;
constexpr int kGradWaves = kGradThreads / 64;
constexpr double kRoot5 = 2.23606797749978969641;
constexpr double kRoot3 = 1.73205080756887729353;
constexpr double kLog2PiD = 1.83787706640934548356;

struct NllArgs {
  const double* X;  // m x d inputs as the covariance sees them (raw when the warp is learned)
  const double* r;  // m_pad: y - c, 0 beyond m
  double* L;        // nb x nb blocks: K, then its lower factor (blocks I >= J)
  double* Xi;       // nb x nb blocks: L^-1 (blocks I >= J)
  double* Di;       // nb blocks: inverses of L's diagonal blocks
  double* Xw;       // m x d warped inputs (warp learned)
  double* Ga;       // m x d: d w / d log a (warp learned)
  double* Gb;       // m x d: d w / d log b (warp learned)
  double* alpha;    // m_pad: K^-1 r
  double* u;        // m_pad: L^-1 r
  double* out;      // [1] 1 when K is numerically positive definite, 0 when not, 2 when a wait ran out
  // Pinned host memory the kernels write their results to: [0] the status of
  // out[1], [1 .. nb] the product of each diagonal block's pivots (real rows),
  // [nb + 1 ..] u (16 nb values), then nb (nb + 1) / 2 x P partial gradient
  // sums (one row per lower block); the host adds them in a fixed order.
  double* hout;
  int m, nb, d, m52, learn_warp;
  double theta[kMaxTheta];
};

// ---- 16 x 16 blocks on the fp64 matrix cores -------------------------------
// v_mfma_f64_16x16x4f64 takes, in lane l (g = l / 16, c = l % 16), A[c][g] and
// B[g][c] of a 16 x 4 by 4 x 16 product and accumulates into a block whose
// register r of lane l is row g + 4r, column c ("C layout").  A 16-deep
// product is four such steps s, with a[s] = A[c][4s + g], b[s] = B[4s + g][c].
__device__ inline d4_t mma16(d4_t acc, const double (&a)[4], const double (&b)[4]) {
#pragma unroll
  for (int s = 0; s < 4; ++s) acc = __builtin_amdgcn_mfma_f64_16x16x4f64(a[s], b[s], acc, 0, 0, 0);
  return acc;
}
// The same from 0 on two chains of two steps, where the result is waited for.
__device__ inline d4_t mma16_zero(const double (&a)[4], const double (&b)[4]) {
  const d4_t z = {0.0, 0.0, 0.0, 0.0};
  d4_t x = __builtin_amdgcn_mfma_f64_16x16x4f64(a[0], b[0], z, 0, 0, 0);
  d4_t y = __builtin_amdgcn_mfma_f64_16x16x4f64(a[1], b[1], z, 0, 0, 0);
  x = __builtin_amdgcn_mfma_f64_16x16x4f64(a[2], b[2], x, 0, 0, 0);
  y = __builtin_amdgcn_mfma_f64_16x16x4f64(a[3], b[3], y, 0, 0, 0);
  return x + y;
}
__device__ inline d4_t zero4() { return d4_t{0.0, 0.0, 0.0, 0.0}; }
// C layout of a row-major block in memory: element 64 r + l.
__device__ inline d4_t ld_c(const double* blk, int lane) {
  return d4_t{blk[lane], blk[64 + lane], blk[128 + lane], blk[192 + lane]};
}
__device__ inline void st_c(double* blk, const d4_t& v, int lane) {
#pragma unroll
  for (int r = 0; r < 4; ++r) blk[64 * r + lane] = v[r];
}
// M[c][4s + g] of a row-major block (A operand from M, B operand from M^T)
__device__ inline void ld_rows(const double* blk, int lane, double (&a)[4]) {
  const double* p = blk + (lane & 15) * 16 + (lane >> 4);
#pragma unroll
  for (int s = 0; s < 4; ++s) a[s] = p[4 * s];
}
// M[4s + g][c] of a row-major block (B operand from M, A operand from M^T): the C layout
__device__ inline void ld_cols(const double* blk, int lane, double (&a)[4]) {
#pragma unroll
  for (int s = 0; s < 4; ++s) a[s] = blk[64 * s + lane];
}
// LDS slots of 256 doubles laid out so that a lane's four operand values are
// contiguous at 4 l: "row slots" hold M[c][4s + g], "column slots" M[4s + g][c].
__device__ inline void ld_slot(const double* slot, int lane, double (&a)[4]) {
  const d2_t* p = reinterpret_cast<const d2_t*>(slot + 4 * lane);
  const d2_t x = p[0], y = p[1];
  a[0] = x[0], a[1] = x[1], a[2] = y[0], a[3] = y[1];
}
// a block in C layout into a column slot (position 4 l + r)
__device__ inline void st_col_slot(double* slot, const d4_t& v, int lane) {
  d2_t* p = reinterpret_cast<d2_t*>(slot + 4 * lane);
  p[0] = d2_t{v[0], v[1]};
  p[1] = d2_t{v[2], v[3]};
}
// position of element (row, col) in a row slot
__device__ inline int row_slot_pos(int row, int col) { return ((col & 3) * 16 + row) * 4 + (col >> 2); }
__device__ inline void st_row_slot(double* slot, const d4_t& v, int lane) {
  const int g = lane >> 4, c = lane & 15;
#pragma unroll
  for (int r = 0; r < 4; ++r) slot[row_slot_pos(g + 4 * r, c)] = v[r];
}

// Next (I, J), J <= I, of a lower triangle enumerated row by row, n steps on.
__device__ inline void advance_lower(int& I, int& J, int n) {
  J += n;
  while (J > I) {
    J -= I + 1;
    ++I;
  }
}

// Lanes of one wave exchanging values through LDS: every LDS access issued
// before has completed (s_waitcnt lgkmcnt(0)) and the compiler moves no memory
// access across.
__device__ inline void wave_lds_sync() {
  asm volatile("" ::: "memory");
  __builtin_amdgcn_s_waitcnt(0xc07f);
  __builtin_amdgcn_wave_barrier();
  asm volatile("" ::: "memory");
}

// Workgroup barrier for waves that exchange data through LDS only: their LDS
// accesses have completed, their global stores may still be in flight.
__device__ inline void lds_barrier() {
  asm volatile("" ::: "memory");
  __builtin_amdgcn_s_waitcnt(0xc07f);
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
}

// Order-fixed sum over the 64 lanes.
__device__ inline double wave_sum(double v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o);
  return v;
}

// The warp of x and its derivatives in log a and log b (0 at x = 0 and 1),
// without cancellation: ln x from log1p(x - 1) above 1/2, 1 - x^a = -expm1(a ln x).
__device__ inline void warp_derivatives(double x, double a, double b, double* w, double* ga, double* gb) {
  x = x < 0.0 ? 0.0 : (x > 1.0 ? 1.0 : x);
  *w = kumaraswamy(x, a, b);
  if (x <= 0.0 || x >= 1.0) {
    *ga = *gb = 0.0;
    return;
  }
  const double lx = x > 0.5 ? log1p(x - 1.0) : log(x);
  const double u = exp(a * lx);
  const double l1u = log(-expm1(a * lx));  // ln(1 - x^a)
  *ga = a * b * exp((b - 1.0) * l1u) * u * lx;
  *gb = -b * exp(b * l1u) * l1u;
}

// Matern covariance at scaled distance t = sqrt(2 nu) r (without tau2).
__device__ inline double matern(bool m52, double s2, double t, double e) {
  return m52 ? s2 * (1.0 + t + t * t / 3.0) * e : s2 * (1.0 + t) * e;
}

// ---- kernel W: warped inputs and their derivatives (warp learned) ---------
__global__ __launch_bounds__(256) void nll_warp_kernel(NllArgs a) {
  const int d = a.d, idx = blockIdx.x * 256 + threadIdx.x;
  if (idx >= a.m * d) return;
  const int k = idx % d;
  warp_derivatives(a.X[idx], exp(a.theta[d + 2 + k]), exp(a.theta[2 * d + 2 + k]), &a.Xw[idx], &a.Ga[idx],
                   &a.Gb[idx]);
}

// ---- kernel K: the covariance, one lower 16 x 16 block per workgroup --------
// Diagonal blocks in full; padding rows and columns are those of the identity.
// Each block is written transposed (column-major), the layout kernel A reads.
__global__ __launch_bounds__(256) void nll_cov_kernel(NllArgs a) {
  __shared__ double sXi[16 * SCOOT_MAX_DIM], sXj[16 * SCOOT_MAX_DIM], sIl[SCOOT_MAX_DIM];
  const int nb = a.nb, m = a.m, d = a.d, t = threadIdx.x;
  int I = 0, J = 0;
  advance_lower(I, J, blockIdx.x);
  const bool m52 = a.m52 != 0;
  const double s2 = exp(a.theta[d]), tau2 = exp(a.theta[d + 1]);
  const double root = m52 ? kRoot5 : kRoot3;
  const double* X = a.learn_warp ? a.Xw : a.X;
  if (t < 16 * d) {
    const int r = t / d, k = t % d, i = 16 * I + r, j = 16 * J + r;
    sXi[t] = i < m ? X[(size_t)i * d + k] : 0.0;
    sXj[t] = j < m ? X[(size_t)j * d + k] : 0.0;
  }
  if (t < d) sIl[t] = exp(-a.theta[t]);
  __syncthreads();
  // block (I, J) is stored transposed: thread t holds element (ii, jj) at t = 16 jj + ii
  const int jj = t >> 4, ii = t & 15, i = 16 * I + ii, j = 16 * J + jj;
  double v;
  if (i < m && j < m) {
    double r2 = 0.0;
    for (int k = 0; k < d; ++k) {
      const double q = (sXi[ii * d + k] - sXj[jj * d + k]) * sIl[k];
      r2 += q * q;
    }
    const double tt = root * sqrt(r2);
    v = matern(m52, s2, tt, exp(-tt)) + (i == j ? tau2 : 0.0);
  } else {
    v = i == j ? 1.0 : 0.0;
  }
  a.L[((size_t)I * nb + J) * 256 + t] = v;
}

// The 64-bit value v of lane src, to every lane (as a scalar).
__device__ inline double lane_bcast(double v, int src) {
  const unsigned long long b = (unsigned long long)__double_as_longlong(v);
  const int lo = __builtin_amdgcn_readlane((int)(unsigned)b, src);
  const int hi = __builtin_amdgcn_readlane((int)(unsigned)(b >> 32), src);
  return __hiloint2double(hi, lo);
}

// 1 / sqrt(p): the hardware estimate r and one third-order step (from the
// series of (1 - e)^-1/2, e = 1 - p r^2: the error is about cubed), a shorter
// dependent chain than two Newton steps or a square root and a division.
__device__ inline double rsqrt_refined(double p) {
  const double r = __builtin_amdgcn_rsq(p);
  const double e = fma(-p * r, r, 1.0);
  return fma(r * e, fma(e, 0.375, 0.5), r);
}

// Factors the 16 x 16 diagonal block kk, held in C layout by one wave, and
// inverts the factor on the way, four columns 4b .. 4b + 3 at a time.  Their
// 4 x 4 diagonal block comes to every lane, which factors it and solves for
// column g (its row group) of the inverse M of that factor.  Rows 4b .. 4b + 3
// of D sit in register b, row 4b + g in group g, where
// v_mfma_f64_16x16x4f64 takes its B operand, and its result's rows 0 .. 3 come
// out the same way in register 0: so one MFMA with M makes four rows of L^T,
// one subtracts their l^T l from the whole block, and two more do the same for
// Y (Y = I at the start, whose rows become those of L^-1).  Bound: one serial
// chain on one wave; with a rank-1 update per column (16 rounds of matrix
// instruction, broadcast, reciprocal root) a block took 6000 cycles, a quarter
// of every round's K = 4 in use; now about 4700, in rounds of four columns.  Stores L_kk column-major to
// memory, L_kk^-1 row-major to memory (Di) and as a row slot (sX), the product
// of the pivots of real rows to sProd[kk]; sets bit 0 of sFlag[0] when such a pivot is
// not above floor (or a padding pivot is not positive).
__device__ inline void diag_factor(const NllArgs& a, int kk, d4_t D, double* sX, double* sProd, int* sFlag,
                                   double floor, int lane) {
  const int g = lane >> 4, j = lane & 15, real = min(16, a.m - 16 * kk);
  d4_t Lt = zero4(), X = zero4(), Y;  // Lt: L^T in C layout (row c of Lt = column c of L)
#pragma unroll
  for (int r = 0; r < 4; ++r) Y[r] = g + 4 * r == j ? 1.0 : 0.0;
  double prod = 1.0;
  bool bad = false;
#pragma unroll
  for (int b = 0; b < 4; ++b) {
    auto at = [&](int r, int c) { return lane_bcast(D[b], r * 16 + 4 * b + c); };
    auto pivot = [&](int r, double p) {
      const bool real_row = 4 * b + r < real;
      bad = bad || !(p > (real_row ? floor : 0.0));
      prod *= real_row ? p : 1.0;
      return rsqrt_refined(p);
    };
    const double i0 = pivot(0, at(0, 0));
    const double l10 = at(1, 0) * i0, l20 = at(2, 0) * i0, l30 = at(3, 0) * i0;
    const double i1 = pivot(1, fma(-l10, l10, at(1, 1)));
    const double l21 = fma(-l20, l10, at(2, 1)) * i1, l31 = fma(-l30, l10, at(3, 1)) * i1;
    const double i2 = pivot(2, fma(-l21, l21, fma(-l20, l20, at(2, 2))));
    const double l32 = fma(-l31, l21, fma(-l30, l20, at(3, 2))) * i2;
    const double i3 = pivot(3, fma(-l32, l32, fma(-l31, l31, fma(-l30, l30, at(3, 3)))));
    // column g of M, then M as an A operand: lane (g, j) holds M[j][g]
    const double y0 = g == 0 ? i0 : 0.0;
    double y1 = fma(-l10, y0, g == 1 ? 1.0 : 0.0) * i1;
    double y2 = fma(-l21, y1, fma(-l20, y0, g == 2 ? 1.0 : 0.0)) * i2;
    double y3 = fma(-l32, y2, fma(-l31, y1, fma(-l30, y0, g == 3 ? 1.0 : 0.0))) * i3;
    asm volatile("" : "+v"(y1), "+v"(y2), "+v"(y3));  // selects below, not branches around the chain
    const double mv = j == 0 ? y0 : (j == 1 ? y1 : (j == 2 ? y2 : (j == 3 ? y3 : 0.0)));
    const d4_t lp = __builtin_amdgcn_mfma_f64_16x16x4f64(mv, D[b], zero4(), 0, 0, 0);
    const double l = j >= 4 * b + g ? lp[0] : 0.0;  // L[j][4b + g], 0 above the diagonal
    Lt[b] = l;
    if (b < 3) D = __builtin_amdgcn_mfma_f64_16x16x4f64(-l, l, D, 0, 0, 0);
    __builtin_amdgcn_sched_barrier(0);  // D, which the next columns wait for, first
    const d4_t yp = __builtin_amdgcn_mfma_f64_16x16x4f64(mv, Y[b], zero4(), 0, 0, 0);
    X[b] = yp[0];                                   // (L^-1)[4b + g][j]
    if (b < 3) Y = __builtin_amdgcn_mfma_f64_16x16x4f64(-l, yp[0], Y, 0, 0, 0);
  }
  st_c(a.L + ((size_t)kk * a.nb + kk) * 256, Lt, lane);  // L_kk column-major
  st_c(a.Di + (size_t)kk * 256, X, lane);
  st_row_slot(sX, X, lane);
  if (lane == 0) {
    sProd[kk] = prod;
    if (bad) __hip_atomic_fetch_or(&sFlag[0], 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
  }
}

// Forward substitution for u = L^-1 r, the diagonal block's part: u_kk =
// L_kk^-1 r_kk with L_kk^-1 from its row slot sX and r_kk (the residual) from
// LDS, as one product C = R L_kk^-T where every row of R is r_kk, so that
// every row of C is u_kk; to sU (16), to memory and to the host.
__device__ inline void diag_solve(const NllArgs& a, int kk, const double* sX, const double* rk, double* sU,
                                  int lane) {
  const int g = lane >> 4, c = lane & 15;
  double av[4], bv[4];
#pragma unroll
  for (int s = 0; s < 4; ++s) av[s] = rk[4 * s + g];
  ld_slot(sX, lane, bv);  // (L_kk^-1)^T as a B operand
  const d4_t v = mma16_zero(av, bv);
  if (lane < 16) {
    sU[c] = v[0];
    a.u[16 * kk + c] = v[0];
    a.hout[1 + a.nb + 16 * kk + c] = v[0];
  }
}

// The residual's update by column k of L: r_i -= L_ik u_k for i = from .. nb - 1,
// with L_ik from its row slot (lane (g, c) holds L_ik[c][4s + g]) and u_k in
// LDS; four blocks at a time, their reads first.
__device__ inline void resid_update(double* sR, const double* pan, const double* uk, int from, int nb, int lane) {
  const int g = lane >> 4;
  const double u[4] = {uk[g], uk[4 + g], uk[8 + g], uk[12 + g]};
  for (int i0 = from; i0 < nb; i0 += 4) {
    double lv[4][4], s[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) ld_slot(pan + (size_t)min(i0 + q, nb - 1) * 256, lane, lv[q]);
#pragma unroll
    for (int q = 0; q < 4; ++q) s[q] = lv[q][0] * u[0] + lv[q][1] * u[1] + lv[q][2] * u[2] + lv[q][3] * u[3];
#pragma unroll
    for (int q = 0; q < 4; ++q) s[q] += __shfl_xor(s[q], 16);
#pragma unroll
    for (int q = 0; q < 4; ++q) s[q] += __shfl_xor(s[q], 32);
    // group q takes block i0 + q
    const double mine = g == 0 ? s[0] : (g == 1 ? s[1] : (g == 2 ? s[2] : s[3]));
    if (i0 + g < nb) sR[16 * i0 + lane] -= mine;
  }
}

// ---- kernel A: the Cholesky factor L and the inverses of its diagonal blocks --
// Blocks are held transposed: the covariance kernel writes block (I, J)
// column-major, the workers' registers hold A_ij^T in C layout (A_ij as an A
// operand), and the factor goes to memory column-major too.  The worker blocks, (i, j) with 1 <= j <= i
// but (1, 1), are listed by decreasing j (then increasing i) and dealt round
// robin to the workers; at step k a worker's blocks with j >= k + 1 form a
// prefix of its share, so each step's work is balanced and the first kRes
// blocks of a share, the longest-lived, stay in registers for the whole
// factorization (the others go through memory each step).
//
// Bound: late steps by wave 0's chain (block update, factor and inverse, about
// 6000 cycles a step), early ones by the workers' updates on three SIMDs'
// matrix units.  m = 256, one launch: 83 us when the workers kept 8 blocks in
// registers, wave 0 took part in every step's barrier and made u as well, and
// a block was factored a column at a time; 67 us now (m = 300: 120 -> 98).  20
// resident blocks are all of a share up to m = 256.  Of the 160,000 cycles
// 19,000 pass before the first step: 280 KB of K come to one CU.
constexpr int kRes = 20;

// f(0), f(1), ... (as constants) until one is false.
template <typename F, int... N>
__device__ inline void while_true(F&& f, std::integer_sequence<int, N...>) {
  (void)(f(std::integral_constant<int, N>()) && ...);
}

__global__ __launch_bounds__(kNllThreads) void nll_factor_kernel(NllArgs a) {
  extern __shared__ __align__(16) double sm[];
  const int nb = a.nb, d = a.d;
  double* sPan = sm;                                // 2 x (nb - 1) row slots: the panels of two columns, rows 1 ..
  double* sX = sPan + (size_t)2 * (nb - 1) * 256;   // 3 row slots: the inverse of diagonal factor k, by k % 3
  double* sDiag = sX + 768;                         // the next diagonal block as updated (column slot)
  double* sOff = sDiag + 256;                       // the block left of it as updated, transposed (column slot)
  double* sProd = sOff + 256;                       // per diagonal block: product of its pivots
  double* sR = sProd + SCOOT_MAX_OBS / 16;          // nb x 16: r, then the forward substitution's residual
  double* sU = sR + (size_t)nb * 16;                // 16: u_k
  // [0] bit 0: a pivot not above its floor, bit 1: a wait ran out; [1] the last
  // diagonal block factored; [2] arrivals at the steps' barriers; [3] blocks
  // handed to wave 0
  int* sFlag = reinterpret_cast<int*>(sU + 16);
  int* sSimd = sFlag + 4;                           // kNllWaves: the SIMD each wave runs on
  int* sList = sSimd + kNllWaves;                   // the worker blocks, (i << 8) | j

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  if (lane == 0) sSimd[wave] = (int)((__builtin_amdgcn_s_getreg((31 << 11) | 4) >> 4) & 3);  // HW_ID.SIMD_ID
  if (tid < 4) sFlag[tid] = tid == 1 ? -1 : 0;
  lds_barrier();

  // Every wait ends: when the flag is there, when something has failed (false),
  // or after a bounded number of looks (false).
  auto flag = [&](int f) { return __hip_atomic_load(&sFlag[f], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP); };
  auto wait = [&](int f, int value) {
    bool alive = true;
    for (int looks = 0;; ++looks) {
      const int now = flag(f), failed = flag(0);
      alive = __builtin_amdgcn_readfirstlane(failed) == 0;
      if (__builtin_amdgcn_readfirstlane(now) >= value || !alive) break;
      if (looks > (1 << 21)) {
        if (lane == 0) __hip_atomic_fetch_or(&sFlag[0], 2, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
        alive = false;
        break;
      }
      __builtin_amdgcn_s_sleep(1);
    }
    wave_lds_sync();
    return alive;
  };
  auto signal = [&](int f) {  // after this wave's LDS writes
    wave_lds_sync();
    if (lane == 0) __hip_atomic_fetch_add(&sFlag[f], 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
  };
  // The n-th barrier (from 1) of all waves but wave 0, which runs ahead.
  auto step_barrier = [&](int n) {
    signal(2);
    return wait(2, (kNllWaves - 1) * n);
  };
  auto panel = [&](int k) { return sPan + ((size_t)(k & 1) * (nb - 1)) * 256 - 256; };  // of column k, by row
  auto inverse = [&](int k) { return sX + (size_t)(k % 3) * 256; };

  // The trailing update goes to the waves that do not share wave 0's SIMD:
  // its vector ALU and the matrix unit are one datapath, so a neighbour's
  // matrix instructions would stall the factorization.
  // One that does (wave 0 itself if there is none) makes u.
  int worker = -1, W = 0, solver = 0;
  for (int w = kNllWaves - 1; w >= 1; --w)
    if (sSimd[w] != sSimd[0]) {
      if (w == wave) worker = W;
      ++W;
    } else {
      solver = w;
    }
  if (W == 0) {  // every wave on one SIMD: all but wave 0 work
    worker = wave - 1;
    W = kNllWaves - 1;
    solver = 0;
  }
  worker = __builtin_amdgcn_readfirstlane(worker);
  W = __builtin_amdgcn_readfirstlane(W);
  solver = __builtin_amdgcn_readfirstlane(solver);
  // a worker's blocks among the first S of the list; the blocks with j >= c
  // are the first (nb - c)(nb - c + 1) / 2 (less (1, 1) when c = 1)
  const unsigned inv_W = 65536u / (unsigned)W + 1;  // x / W = x inv_W >> 16 for the list's x < 2^10
  auto mine_below = [&](int S) { return S > worker ? (int)(((unsigned)(S - 1 - worker) * inv_W) >> 16) + 1 : 0; };
  auto from_col = [&](int c) { return (nb - c) * (nb - c + 1) / 2 - (c <= 1 ? 1 : 0); };
  auto solve = [&](int k) {  // u_k
    diag_solve(a, k, inverse(k), sR + 16 * k, sU, lane);
    wave_lds_sync();
  };
  auto solve_step = [&](int k) {
    solve(k);
    resid_update(sR, panel(k), sU, k + 1, nb, lane);
    wave_lds_sync();
  };
  if (wave == solver) {
    for (int i = lane; i < nb * 16; i += 64) sR[i] = a.r[i];
    wave_lds_sync();
  }

  // ---- Cholesky factor, 16 columns per step --------------------------------
  // Before step k the panel of column k, L_ik (i > k), is in row slots and
  // L_kk^-1 in sX.  Step k: the workers apply column k to their blocks with
  // j >= k+1, A_ij^T -= L_jk L_ik^T, hand blocks (k+2, k+2) and (k+2, k+1) to
  // wave 0 through LDS, and once wave 0 has published the new inverse turn
  // their blocks of column k+1 into the panel,
  // L_i,k+1^T = L_k+1,k+1^-1 A_i,k+1^T; the solver takes u_k = L_kk^-1 r_k and
  // column k's term off the residuals below.  Wave 0 makes L_k+1,k for itself
  // from the blocks handed over one step earlier, applies it to block
  // (k+1, k+1), factors and inverts that block, takes the next two blocks and
  // publishes the inverse; so it never waits for a panel, and the workers'
  // writes of a step (after the previous inverse) meet no read of the
  // step before.  An inverse is read by the solver one step later, while wave
  // 0 may be one step ahead: three slots.  The waves share data through LDS
  // only (a worker reads back only blocks it wrote), so no wait covers global
  // stores.  Every role has a loop of its own, so that the workers' resident
  // blocks hold no registers where wave 0 factors.
  if (wave == 0) {
    const double s2 = exp(a.theta[d]), tau2 = exp(a.theta[d + 1]);
    // A pivot that is not above 1e-13 of its original diagonal entry (s2 + tau2)
    // means K is not numerically positive definite (the host factor's rule).
    const double floor = 1e-13 * (s2 + tau2);
    d4_t D = ld_c(a.L, lane), Dn = zero4();
    double off[4] = {0.0, 0.0, 0.0, 0.0};
    if (nb > 1) {  // blocks (1, 1) and (1, 0): the covariance itself
      Dn = ld_c(a.L + ((size_t)nb + 1) * 256, lane);
      ld_cols(a.L + (size_t)nb * 256, lane, off);
    }
    // both here before the first inverse is published: the workers then write
    // the panel over block (1, 0)
    asm volatile("" : "+v"(Dn), "+v"(off[0]), "+v"(off[1]), "+v"(off[2]), "+v"(off[3]));
    bool alive = true;
    for (int k = 0; k < nb && alive; ++k) {
      diag_factor(a, k, D, inverse(k), sProd, sFlag, floor, lane);
      if (k >= 1 && k + 1 < nb) {  // blocks (k+1, k+1) and (k+1, k), column k-1 applied
        alive = wait(3, 2 * k);
        double dv[4];
        ld_slot(sDiag, lane, dv);
        ld_slot(sOff, lane, off);
        Dn = d4_t{dv[0], dv[1], dv[2], dv[3]};
      }
      wave_lds_sync();  // the inverse is in LDS, the blocks are read
      if (lane == 0) __hip_atomic_store(&sFlag[1], k, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
      if (k + 1 < nb) {
        double xv[4];
        ld_slot(inverse(k), lane, xv);
        const d4_t v = mma16_zero(xv, off);  // L_k+1,k^T: both operands of its product as it stands
        const double av[4] = {-v[0], -v[1], -v[2], -v[3]}, bv[4] = {v[0], v[1], v[2], v[3]};
        D = Dn + mma16_zero(av, bv);
        if (solver == 0) {
          alive = wait(2, (kNllWaves - 1) * (k + 1)) && alive;  // the panel of column k is made
          solve_step(k);
        }
      }
    }
  } else {
    constexpr int kCol0 = (SCOOT_MAX_OBS / 16 - 1 + kNllWaves - 2) / (kNllWaves - 1);  // column-0 blocks per wave
    double c0[kCol0][4];
    d4_t res[kRes];  // a worker's first kRes blocks (transposed, C layout)
    unsigned rij[kRes / 2];  // their (i << 8) | j, two to a register
    const int n_list = nb > 1 ? nb * (nb - 1) / 2 - 1 : 0;
    const int n_share = worker >= 0 ? mine_below(n_list) : 0;
    // while wave 0 factors block (0, 0): column 0, the list, the resident blocks
#pragma unroll
    for (int t = 0; t < kCol0; ++t) {
      const int i = wave + (kNllWaves - 1) * t;
      if (i < nb) ld_cols(a.L + (size_t)i * nb * 256, lane, c0[t]);  // A_i0^T as a B operand
    }
    int first = (1 << 8) | 1;  // lane e: the worker's entry e < 64 (a block that exists, past its share)
    for (int e = lane; e < n_share; e += 64) {  // the worker's own entries
      int n = worker + W * e;
      for (int j = nb - 1; j >= 1; --j) {
        const int lo = j == 1 ? 2 : j, cnt = nb - lo;
        if (n < cnt) {
          sList[worker + W * e] = ((lo + n) << 8) | j;
          if (e == lane) first = ((lo + n) << 8) | j;
          break;
        }
        n -= cnt;
      }
    }
    auto entry = [&](int e) {
      return e < 64 ? __builtin_amdgcn_readlane(first, e) : __builtin_amdgcn_readfirstlane(sList[worker + W * e]);
    };
#pragma unroll
    for (int s = 0; s < kRes; ++s) {
      const int ij = __builtin_amdgcn_readlane(first, s);
      rij[s / 2] = s & 1 ? rij[s / 2] | (unsigned)ij << 16 : (unsigned)ij;
      res[s] = zero4();
      if (s < n_share) res[s] = ld_c(a.L + ((size_t)(ij >> 8) * nb + (ij & 255)) * 256, lane);
    }
    // all here: a register with a load in flight would make every later use of
    // it, in the loop too, wait for the stores issued since
    __builtin_amdgcn_s_waitcnt(0x0f70);
    // the panel of column 0: L_i0^T = L_00^-1 A_i0^T (C layout, so column-major
    // to memory and a row slot of L_i0 as it stands)
    wait(1, 0);
    {
      double xv[4];
      ld_slot(inverse(0), lane, xv);
#pragma unroll
      for (int t = 0; t < kCol0; ++t) {
        const int i = wave + (kNllWaves - 1) * t;
        if (i < nb) {
          const d4_t v = mma16_zero(xv, c0[t]);
          st_c(a.L + (size_t)i * nb * 256, v, lane);
          st_col_slot(panel(0) + (size_t)i * 256, v, lane);
        }
      }
    }
    bool alive = step_barrier(1);
    for (int k = 0; k + 1 < nb && alive; ++k) {
      if (wave == solver) solve_step(k);
      const double* pc = panel(k);
      double* pn = panel(k + 1);  // being made
      const int n_trail = worker >= 0 ? mine_below(from_col(k + 2)) : 0;  // the share's blocks with j >= k+2
      const int n_act = worker >= 0 ? mine_below(from_col(k + 1)) : 0;    // ... with j >= k+1
      // block (k+2, k+2), the first of its column, is entry e_diag of the share
      const int at_diag = from_col(k + 3) - worker;
      const int e_diag = k + 2 < nb && at_diag >= 0 && (mine_below(from_col(k + 3) + 1) - 1) * W == at_diag
                             ? mine_below(from_col(k + 3) + 1) - 1 : -1;
      // Updated block e of the share: those of column k+1 wait in the new
      // panel's slots, (k+2, k+2) and (k+2, k+1) go to wave 0 as well.
      auto updated = [&](int e, int i, const d4_t& v) {
        if (e >= n_trail && e < n_act && i > k + 1) {
          st_col_slot(pn + (size_t)i * 256, v, lane);
          if (i == k + 2) {
            st_col_slot(sOff, v, lane);
            signal(3);
          }
        }
        if (e == e_diag) {
          st_col_slot(sDiag, v, lane);
          signal(3);
        }
      };
      // resident blocks, two at a time (block (k+1, k+1) and a block that has
      // died are updated to no effect); the first pair past the share ends it,
      // so that a late step does not step over every dead pair
      auto update_pair = [&](auto pair) {
        constexpr int s = 2 * decltype(pair)::value;
        if (s >= n_act) return false;
        double av[2][4], bv[2][4];
#pragma unroll
        for (int u = 0; u < 2; ++u) {
          ld_slot(pc + (size_t)((rij[s / 2] >> (16 * u)) & 255) * 256, lane, av[u]);
          ld_slot(pc + (size_t)((rij[s / 2] >> (16 * u + 8)) & 255) * 256, lane, bv[u]);
        }
#pragma unroll
        for (int q = 0; q < 4; ++q)
#pragma unroll
          for (int u = 0; u < 2; ++u)
            res[s + u] = __builtin_amdgcn_mfma_f64_16x16x4f64(-av[u][q], bv[u][q], res[s + u], 0, 0, 0);
        if (s + 1 >= n_trail || s == (e_diag & ~1)) {
#pragma unroll
          for (int u = 0; u < 2; ++u) updated(s + u, (rij[s / 2] >> (16 * u + 8)) & 255, res[s + u]);
        }
        __builtin_amdgcn_sched_barrier(0);  // a block's operands loaded where it is updated
        return true;
      };
      while_true(update_pair, std::make_integer_sequence<int, kRes / 2>());
      // the others, four at a time, their loads first; the blocks with
      // j >= k+2 go back to memory
      for (int e0 = kRes; e0 < n_act; e0 += 4) {
        d4_t acc[4];
        int ij[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          ij[u] = entry(e0 + u < n_act ? e0 + u : e0);
          acc[u] = ld_c(a.L + ((size_t)(ij[u] >> 8) * nb + (ij[u] & 255)) * 256, lane);
        }
        // all four here, used or not: registers with a load in flight would make
        // later code wait for every store too
        __builtin_amdgcn_s_waitcnt(0x0f70);
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          const int i = ij[u] >> 8, j = ij[u] & 255;
          if (e0 + u < n_act) {
            double av[4], bv[4];
            ld_slot(pc + (size_t)j * 256, lane, av);
            ld_slot(pc + (size_t)i * 256, lane, bv);
#pragma unroll
            for (int q = 0; q < 4; ++q) av[q] = -av[q];
            acc[u] = mma16(acc[u], av, bv);
            if (e0 + u < n_trail) st_c(a.L + ((size_t)i * nb + j) * 256, acc[u], lane);
            updated(e0 + u, i, acc[u]);
          }
        }
      }
      // the panel of column k+1, two blocks at a time, the blocks' own reads
      // before the wait for the inverse
      double xv[4];
      bool have_x = false;
      for (int e = n_trail; e < n_act; e += 2) {
        const int i0 = entry(e) >> 8, i1 = entry(e + 1 < n_act ? e + 1 : e) >> 8;
        double t0[4], t1[4];
        ld_slot(pn + (size_t)i0 * 256, lane, t0);
        ld_slot(pn + (size_t)i1 * 256, lane, t1);
        if (!have_x) {
          if (i0 == k + 1 && (e + 1 == n_act || i1 == k + 1)) continue;  // block (k+1, k+1) alone
          wait(1, k + 1);
          ld_slot(inverse(k + 1), lane, xv);
          have_x = true;
        }
        const d4_t v0 = mma16_zero(xv, t0), v1 = mma16_zero(xv, t1);
        if (i0 != k + 1) {
          st_col_slot(pn + (size_t)i0 * 256, v0, lane);
          st_c(a.L + ((size_t)i0 * nb + k + 1) * 256, v0, lane);
        }
        if (i1 != i0) {
          st_col_slot(pn + (size_t)i1 * 256, v1, lane);
          st_c(a.L + ((size_t)i1 * nb + k + 1) * 256, v1, lane);
        }
      }
      alive = step_barrier(k + 2);
    }
  }
  if (wave == solver) {
    if (wait(1, nb - 1)) solve(nb - 1);
  }
  lds_barrier();  // all waves
  // status: 1 factored, 0 not positive definite, 2 a wait ran out (reported as
  // a device failure)
  const int failed = flag(0);
  const double status = (failed & 2) ? 2.0 : (failed ? 0.0 : 1.0);
  if (tid == 0) {
    a.out[1] = status;
    a.hout[0] = status;
  }
  if (status == 1.0 && tid < nb) a.hout[1 + tid] = sProd[tid];
}

// ---- kernel T: L^-1, one block column per workgroup ---------------------------
// Column j: X_jj = Di_j, and for i > j
//   X_ij = -Di_i S_ij,   S_ij = sum_{k=j}^{i-1} L_ik X_kj.
// Right-looking: as soon as X_kj is known every later row i adds its term
// L_ik X_kj to S_ij, which the wave that finishes row i keeps in registers
// (rows dealt round robin to the waves, R per wave at most); the owner of row
// k+1 then finishes X_k+1,j into LDS, where the column stays until it is
// written out at the end.  L was written by another compute unit, so its
// blocks (column-major: an A operand is a contiguous read) are loaded
// kTriAhead steps ahead into a ring of registers, and Di up front; every step
// issues the same loads (a row with nothing to load reads block (0, 0)), so
// each wait is for exactly the load it needs.
constexpr int kTriWaves = 8;
constexpr int kTriMaxRows = (SCOOT_MAX_OBS / 16 - 1 + kTriWaves - 1) / kTriWaves;
constexpr int kTriAhead = 3;

template <int R>
struct TriState {
  d4_t S[R];
  double Lv[kTriAhead][R][4];  // ring: L_ik for steps k, k+1, k+2 in slot (k - j) % 3
  double Dv[R][4];             // Di_i
};

// Step k of column j; ring slot B holds L_ik.  Steps past the column's end
// only load and wait, so that every wave runs the same number of barriers.
template <int R, int B>
__device__ inline void tri_step(const NllArgs& a, TriState<R>& st, double* sXcol, int j, int k, int wave,
                                int lane) {
  const int nb = a.nb;
  double xv[4];
  ld_slot(sXcol + (size_t)(k < nb ? k : nb - 1) * 256, lane, xv);  // X_kj as a B operand
#pragma unroll
  for (int t = 0; t < R; ++t) {
    const int i = j + 1 + wave + kTriWaves * t;
    if (i > k && i < nb) {  // row k+1 (if this wave's) comes first
      st.S[t] = mma16(st.S[t], st.Lv[B][t], xv);
      if (i == k + 1) {
        double nd[4];
#pragma unroll
        for (int s = 0; s < 4; ++s) nd[s] = -st.Dv[t][s];
        const double sv[4] = {st.S[t][0], st.S[t][1], st.S[t][2], st.S[t][3]};  // S as a B operand is its own C layout
        st_col_slot(sXcol + (size_t)i * 256, mma16(zero4(), nd, sv), lane);
      }
    }
    const bool next = i < nb && k + kTriAhead < i;
    ld_cols(a.L + (next ? ((size_t)i * nb + k + kTriAhead) * 256 : 0), lane, st.Lv[B][t]);
  }
  lds_barrier();
}

template <int R>
__global__ __launch_bounds__(kTriWaves * 64) void nll_trtri_kernel(NllArgs a) {
  extern __shared__ __align__(16) double sXcol[];  // nb column slots: X_ij, i >= j
  if (a.out[1] != 1.0) return;
  double* sAl = sXcol + (size_t)a.nb * 256;        // kTriWaves x 16: alpha's parts
  const int nb = a.nb, j = blockIdx.x, lane = threadIdx.x & 63, g = lane >> 4;
  const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
  TriState<R> st;
  // u_i[4s + g] of the wave's rows and of row j (wave 0), loaded up front
  // unless the registers are wanted for the ring
  double uv[R + 1][4];
  auto load_u = [&]() {
#pragma unroll
    for (int t = 0; t <= R; ++t) {
      const int i = t < R ? j + 1 + wave + kTriWaves * t : j;
#pragma unroll
      for (int s = 0; s < 4; ++s) uv[t][s] = i < nb ? a.u[16 * i + 4 * s + g] : 0.0;
    }
  };
  if constexpr (R <= 4) load_u();
#pragma unroll
  for (int t = 0; t < R; ++t) {
    st.S[t] = zero4();
    const int i = j + 1 + wave + kTriWaves * t;
#pragma unroll
    for (int b = 0; b < kTriAhead; ++b)
      ld_cols(a.L + (i < nb && j + b < i ? ((size_t)i * nb + j + b) * 256 : 0), lane, st.Lv[b][t]);
    ld_rows(a.Di + (i < nb ? (size_t)i * 256 : 0), lane, st.Dv[t]);
  }
  if (wave == 0) st_col_slot(sXcol + (size_t)j * 256, ld_c(a.Di + (size_t)j * 256, lane), lane);
  // all of the above in registers before the loop, so that inside it a wait
  // is only ever for the ring slot about to be used
  __builtin_amdgcn_s_waitcnt(0);
  lds_barrier();
  for (int k = j; k + 1 < nb; k += kTriAhead) {
    tri_step<R, 0>(a, st, sXcol, j, k, wave, lane);
    tri_step<R, 1>(a, st, sXcol, j, k + 1, wave, lane);
    tri_step<R, 2>(a, st, sXcol, j, k + 2, wave, lane);
  }
  // the column, row-major blocks
  for (int i = j + wave; i < nb; i += kTriWaves) {
    double x[4];
    ld_slot(sXcol + (size_t)i * 256, lane, x);
    st_c(a.Xi + ((size_t)i * nb + j) * 256, d4_t{x[0], x[1], x[2], x[3]}, lane);
  }
  // alpha_j = sum_{i >= j} X_ij^T u_i (alpha = L^-T L^-1 r): each wave its rows,
  // then the waves in order
  if constexpr (R > 4) load_u();
  double acc = 0.0;
#pragma unroll
  for (int t = 0; t <= R; ++t) {
    const int i = t < R ? j + 1 + wave + kTriWaves * t : j;
    if (i < nb && (t < R || wave == 0)) {
      double x[4];
      ld_slot(sXcol + (size_t)i * 256, lane, x);  // X_ij[4s + g][c]
#pragma unroll
      for (int s = 0; s < 4; ++s) acc = fma(x[s], uv[t][s], acc);
    }
  }
  acc += __shfl_xor(acc, 16);
  acc += __shfl_xor(acc, 32);
  if (lane < 16) sAl[wave * 16 + lane] = acc;
  lds_barrier();
  if (wave == 0 && lane < 16) {
    double s = 0.0;
#pragma unroll
    for (int w = 0; w < kTriWaves; ++w) s += sAl[w * 16 + lane];
    a.alpha[16 * j + lane] = s;
  }
}

// ---- kernel B: the gradient's partial sums, one lower block per workgroup ---
// Z_IJ = (K^-1)_IJ = sum_{k >= I} X_kI^T X_kJ on the matrix cores (wave w
// takes k = I + w, I + w + 4, ...; the four sums are added in order through
// LDS, and a diagonal block is made exactly symmetric), then one element of
// W = alpha alpha^T - K^-1 per thread with the covariance and its
// derivatives recomputed.
template <int D, bool LW>
__global__ __launch_bounds__(kGradThreads) void nll_grad_kernel(NllArgs a) {
  constexpr int P = LW ? 3 * D + 2 : D + 2;
  __shared__ double sZ[kGradWaves][256];
  __shared__ double sRed[kGradWaves][P];
  if (a.out[1] != 1.0) return;  // K not positive definite: no gradient
  const int nb = a.nb, m = a.m, t = threadIdx.x, lane = t & 63, wave = t >> 6;
  int I = 0, J = 0;
  advance_lower(I, J, blockIdx.x);
  d4_t Zv = zero4();
  for (int k0 = I + wave; k0 < nb; k0 += 4 * kGradWaves) {
    double av[4][4], bv[4][4];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int k = k0 + u * kGradWaves;
      if (k < nb) {
        ld_cols(a.Xi + ((size_t)k * nb + I) * 256, lane, av[u]);  // X_kI^T as an A operand
        ld_cols(a.Xi + ((size_t)k * nb + J) * 256, lane, bv[u]);  // X_kJ as a B operand
      }
    }
#pragma unroll
    for (int u = 0; u < 4; ++u)
      if (k0 + u * kGradWaves < nb) Zv = mma16(Zv, av[u], bv[u]);
  }
  st_c(sZ[wave], Zv, lane);
  __syncthreads();
  const int ii = t >> 4, jj = t & 15, i = 16 * I + ii, j = 16 * J + jj;
  double zij = ((sZ[0][t] + sZ[1][t]) + sZ[2][t]) + sZ[3][t];
  if (I == J) {
    const int tt = jj * 16 + ii;
    zij = 0.5 * (zij + (((sZ[0][tt] + sZ[1][tt]) + sZ[2][tt]) + sZ[3][tt]));
  }
  double g[P];
#pragma unroll
  for (int p = 0; p < P; ++p) g[p] = 0.0;
  if (!((I == J && jj > ii) || i >= m || j >= m)) {
    const bool m52 = a.m52 != 0;
    const double s2 = exp(a.theta[D]), tau2 = exp(a.theta[D + 1]);
    const double root = m52 ? kRoot5 : kRoot3;
    const double* X = LW ? a.Xw : a.X;
    const double w = 0.5 * (i == j ? 1.0 : 2.0) * (a.alpha[i] * a.alpha[j] - zij);  // W and dK are symmetric
    double tk[D], inv_ls[D], r2 = 0.0;
#pragma unroll
    for (int k = 0; k < D; ++k) {
      inv_ls[k] = exp(-a.theta[k]);
      tk[k] = (X[(size_t)i * D + k] - X[(size_t)j * D + k]) * inv_ls[k];
      r2 += tk[k] * tk[k];
    }
    const double tt = root * sqrt(r2), e = exp(-tt);
    const double kv = matern(m52, s2, tt, e);
    const double rad = m52 ? 5.0 / 3.0 * s2 * (1.0 + tt) * e : 3.0 * s2 * e;
    const double wr = w * rad;
#pragma unroll
    for (int k = 0; k < D; ++k) {
      g[k] -= wr * (tk[k] * tk[k]);
      if constexpr (LW) {
        const double wt = wr * tk[k] * inv_ls[k];
        g[D + 2 + k] += wt * (a.Ga[(size_t)i * D + k] - a.Ga[(size_t)j * D + k]);
        g[2 * D + 2 + k] += wt * (a.Gb[(size_t)i * D + k] - a.Gb[(size_t)j * D + k]);
      }
    }
    g[D] -= w * kv;
    if (i == j) g[D + 1] -= w * tau2;
  }
#pragma unroll
  for (int p = 0; p < P; ++p) {
    const double v = wave_sum(g[p]);
    if (lane == 0) sRed[wave][p] = v;
  }
  __syncthreads();
  if (t < P) {
    double s = 0.0;
#pragma unroll
    for (int w = 0; w < kGradWaves; ++w) s += sRed[w][t];
    a.hout[1 + 17 * nb + (size_t)blockIdx.x * P + t] = s;
  }
}

template <int D, typename F>
int by_dim(int d, F&& f) {
  if constexpr (D > SCOOT_MAX_DIM) {
    return fail(SCOOT_ERR_UNSUPPORTED, "gp nll: d exceeds SCOOT_MAX_DIM");
  } else {
    if (d == D) return f(std::integral_constant<int, D>());
    return by_dim<D + 1>(d, std::forward<F>(f));
  }
}

// Device state of one likelihood (one objective): inputs, work matrices and a
// pinned read-back buffer, all allocated once per search.
class DeviceNll {
 public:
  ~DeviceNll() {
    if (buf_) (void)hipFree(buf_);
    if (host_) (void)hipHostFree(host_);
  }
  int init(const std::vector<double>& X, const std::vector<double>& r, int m, int d, scoot_kernel kernel,
           bool learn_warp, hipStream_t s) {
    s_ = s;
    m_ = m;
    d_ = d;
    lw_ = learn_warp;
    P_ = learn_warp ? 3 * d + 2 : d + 2;
    nb_ = (m + 15) / 16;
    // every part 256-byte aligned (32 doubles)
    auto up = [](size_t n) { return (n + 31) / 32 * 32; };
    const size_t md = (size_t)m * d, mp = (size_t)nb_ * 16, blocks = (size_t)nb_ * nb_ * 256;
    const size_t n = up(md) + up(mp) + 2 * blocks + (size_t)nb_ * 256 + (learn_warp ? 3 * up(md) : 0) +
                     2 * up(mp) + up(2);
    if (hipMalloc(&buf_, n * sizeof(double)) != hipSuccess) {
      buf_ = nullptr;
      return fail(SCOOT_ERR_NO_MEMORY, "gp nll: device allocation failed");
    }
    // the results, written by the kernels straight into coherent pinned host
    // memory (no copy after them): status, pivot products, u, partial gradient
    // sums
    n_lower_ = nb_ * (nb_ + 1) / 2;
    if (hipHostMalloc(&host_, (1 + 17 * (size_t)nb_ + (size_t)n_lower_ * P_) * sizeof(double),
                      hipHostMallocMapped | hipHostMallocCoherent) != hipSuccess) {
      host_ = nullptr;
      return fail(SCOOT_ERR_NO_MEMORY, "gp nll: pinned allocation failed");
    }
    void* hdev = nullptr;
    if (hipHostGetDevicePointer(&hdev, host_, 0) != hipSuccess || hdev == nullptr)
      return fail(SCOOT_ERR_DEVICE, "gp nll: pinned memory not visible to the device");
    a_.hout = static_cast<double*>(hdev);
    double* p = buf_;
    double* Xd = p;
    p += up(md);
    double* rd = p;
    p += up(mp);
    a_.L = p;
    p += blocks;
    a_.Xi = p;
    p += blocks;
    a_.Di = p;
    p += (size_t)nb_ * 256;
    a_.Xw = a_.Ga = a_.Gb = nullptr;
    if (learn_warp) {
      a_.Xw = p;
      a_.Ga = p + up(md);
      a_.Gb = p + 2 * up(md);
      p += 3 * up(md);
    }
    a_.alpha = p;
    p += up(mp);
    a_.u = p;
    p += up(mp);
    a_.out = p;
    a_.X = Xd;
    a_.r = rd;
    a_.m = m;
    a_.nb = nb_;
    a_.d = d;
    a_.m52 = kernel == SCOOT_MATERN52;
    a_.learn_warp = learn_warp;
    std::vector<double> rp(mp, 0.0);
    std::memcpy(rp.data(), r.data(), sizeof(double) * m);
    if (hipMemcpyAsync(Xd, X.data(), md * sizeof(double), hipMemcpyHostToDevice, s) != hipSuccess ||
        hipMemcpyAsync(rd, rp.data(), mp * sizeof(double), hipMemcpyHostToDevice, s) != hipSuccess ||
        hipStreamSynchronize(s) != hipSuccess)
      return fail(SCOOT_ERR_DEVICE, std::string("gp nll: upload failed: ") + hipGetErrorString(hipGetLastError()));
    lds_ = ((size_t)(nb_ - 1) * 512 + 768 + 512 + SCOOT_MAX_OBS / 16 + (size_t)nb_ * 16 + 16) * sizeof(double) +
           (4 + kNllWaves + (size_t)nb_ * (nb_ - 1) / 2) * sizeof(int);

    int rc = allow_full_lds((const void*)nll_factor_kernel, "gp nll");
    const void* tri[] = {(const void*)nll_trtri_kernel<1>, (const void*)nll_trtri_kernel<2>,
                         (const void*)nll_trtri_kernel<3>, (const void*)nll_trtri_kernel<4>,
                         (const void*)nll_trtri_kernel<kTriMaxRows>};
    for (const void* f : tri)
      if (rc == SCOOT_OK) rc = allow_full_lds(f, "gp nll");
    return rc;
  }
  // false when K is not positive definite; a device failure is kept in error().
  bool eval(const double* theta, double* nll, double* grad) {
    if (rc_ != SCOOT_OK) return false;
    std::memcpy(a_.theta, theta, sizeof(double) * P_);
    (void)hipGetLastError();  // clear an earlier, unrelated error
    if (lw_)
      hipLaunchKernelGGL(nll_warp_kernel, dim3((unsigned)((m_ * d_ + 255) / 256)), dim3(256), 0, s_, a_);
    hipLaunchKernelGGL(nll_cov_kernel, dim3((unsigned)(nb_ * (nb_ + 1) / 2)), dim3(256), 0, s_, a_);
    hipLaunchKernelGGL(nll_factor_kernel, dim3(1), dim3(kNllThreads), lds_, s_, a_);
    if (grad) {  // L^-1 and alpha, then K^-1 and the gradient's partial sums (the NLL needs none of them)
      launch_trtri();
      const int rc = by_dim<1>(d_, [&](auto D) {
        if (lw_)
          hipLaunchKernelGGL((nll_grad_kernel<decltype(D)::value, true>), dim3((unsigned)n_lower_), dim3(kGradThreads), 0,
                             s_, a_);
        else
          hipLaunchKernelGGL((nll_grad_kernel<decltype(D)::value, false>), dim3((unsigned)n_lower_), dim3(kGradThreads), 0,
                             s_, a_);
        return SCOOT_OK;
      });
      if (rc != SCOOT_OK) {
        rc_ = rc;
        return false;
      }
    }
    const hipError_t launched = hipGetLastError();
    if (launched != hipSuccess) {
      rc_ = fail(SCOOT_ERR_DEVICE, std::string("gp nll: launch failed: ") + hipGetErrorString(launched));
      return false;
    }
    if (hipStreamSynchronize(s_) != hipSuccess) {
      rc_ = fail(SCOOT_ERR_DEVICE, std::string("gp nll: device evaluation failed: ") +
                                       hipGetErrorString(hipGetLastError()));
      return false;
    }
    if (host_[0] == 2.0) {
      rc_ = fail(SCOOT_ERR_DEVICE, "gp nll: the factorization's wait for its diagonal block ran out");
      return false;
    }
    if (host_[0] != 1.0) return false;
    // NLL = 1/2 |L^-1 r|^2 + 1/2 log det K + m/2 log(2 pi), and the gradient's
    // partial sums, each added in a fixed order
    double q = 0.0, logdet = 0.0;
    for (int k = 0; k < nb_; ++k) logdet += std::log(host_[1 + k]);
    for (int i = 0; i < 16 * nb_; ++i) q += host_[1 + nb_ + i] * host_[1 + nb_ + i];
    *nll = 0.5 * q + 0.5 * logdet + 0.5 * m_ * kLog2PiD;
    if (grad) {
      const double* part = host_ + 1 + 17 * nb_;
      for (int p = 0; p < P_; ++p) {
        double s = 0.0;
        for (int b = 0; b < n_lower_; ++b) s += part[(size_t)b * P_ + p];
        grad[p] = s;
      }
    }
    return true;
  }
  // K, the factor, L^-1 and alpha at theta, launched.
  bool launch_factor(const double* theta) {
    if (rc_ != SCOOT_OK) return false;
    std::memcpy(a_.theta, theta, sizeof(double) * P_);
    (void)hipGetLastError();  // clear an earlier, unrelated error
    if (lw_)
      hipLaunchKernelGGL(nll_warp_kernel, dim3((unsigned)((m_ * d_ + 255) / 256)), dim3(256), 0, s_, a_);
    hipLaunchKernelGGL(nll_cov_kernel, dim3((unsigned)(nb_ * (nb_ + 1) / 2)), dim3(256), 0, s_, a_);
    hipLaunchKernelGGL(nll_factor_kernel, dim3(1), dim3(kNllThreads), lds_, s_, a_);
    launch_trtri();
    const hipError_t launched = hipGetLastError();
    if (launched != hipSuccess) {
      rc_ = fail(SCOOT_ERR_DEVICE, std::string("gp fit: launch failed: ") + hipGetErrorString(launched));
      return false;
    }
    return true;
  }
  // After a synchronisation: false when K is not positive definite or on a
  // device failure (kept in error()).
  bool factored() {
    if (host_[0] == 2.0) {
      rc_ = fail(SCOOT_ERR_DEVICE, "gp fit: the factorization's wait for its diagonal block ran out");
      return false;
    }
    return host_[0] == 1.0;
  }
  const double* Xi() const { return a_.Xi; }
  const double* alpha() const { return a_.alpha; }
  int blocks() const { return nb_; }
  hipStream_t stream() const { return s_; }
  // launch_factor, then L^-1 (m x m row-major, lower) and alpha to the host;
  // false when K is not positive definite or on a device failure.
  bool inverse(const double* theta, std::vector<double>& Linv, std::vector<double>& alpha) {
    if (!launch_factor(theta)) return false;
    if (hipStreamSynchronize(s_) != hipSuccess) {
      rc_ = fail(SCOOT_ERR_DEVICE, std::string("gp fit: device factorization failed: ") +
                                       hipGetErrorString(hipGetLastError()));
      return false;
    }
    if (!factored()) return false;
    std::vector<double> xi((size_t)nb_ * nb_ * 256), al((size_t)nb_ * 16);
    if (hipMemcpyAsync(xi.data(), a_.Xi, xi.size() * sizeof(double), hipMemcpyDeviceToHost, s_) != hipSuccess ||
        hipMemcpyAsync(al.data(), a_.alpha, al.size() * sizeof(double), hipMemcpyDeviceToHost, s_) != hipSuccess ||
        hipStreamSynchronize(s_) != hipSuccess) {
      rc_ = fail(SCOOT_ERR_DEVICE, std::string("gp fit: read-back failed: ") + hipGetErrorString(hipGetLastError()));
      return false;
    }
    const int m = m_;
    Linv.assign((size_t)m * m, 0.0);
    for (int row = 0; row < m; ++row)
      for (int col = 0; col <= row; ++col) {
        const int I = row >> 4, J = col >> 4;
        Linv[(size_t)row * m + col] = xi[((size_t)I * nb_ + J) * 256 + (row & 15) * 16 + (col & 15)];
      }
    alpha.assign(al.begin(), al.begin() + m);
    return true;
  }
  int error() const { return rc_; }

 private:
  void launch_trtri() {
    const size_t lds_tri = ((size_t)nb_ * 256 + kTriWaves * 16) * sizeof(double);
    switch ((nb_ - 1 + kTriWaves - 1) / kTriWaves) {
      case 0:
      case 1: hipLaunchKernelGGL(nll_trtri_kernel<1>, dim3((unsigned)nb_), dim3(kTriWaves * 64), lds_tri, s_, a_); break;
      case 2: hipLaunchKernelGGL(nll_trtri_kernel<2>, dim3((unsigned)nb_), dim3(kTriWaves * 64), lds_tri, s_, a_); break;
      case 3: hipLaunchKernelGGL(nll_trtri_kernel<3>, dim3((unsigned)nb_), dim3(kTriWaves * 64), lds_tri, s_, a_); break;
      case 4: hipLaunchKernelGGL(nll_trtri_kernel<4>, dim3((unsigned)nb_), dim3(kTriWaves * 64), lds_tri, s_, a_); break;
      default: hipLaunchKernelGGL(nll_trtri_kernel<kTriMaxRows>, dim3((unsigned)nb_), dim3(kTriWaves * 64), lds_tri, s_, a_);
    }
  }
  hipStream_t s_ = nullptr;
  int m_ = 0, d_ = 0, nb_ = 0, n_lower_ = 0, P_ = 0;
  bool lw_ = false;
  size_t lds_ = 0;
  double* buf_ = nullptr;
  double* host_ = nullptr;
  NllArgs a_{};
  int rc_ = SCOOT_OK;
};

int device_inputs(const double* X, const double* y, int m, int d, scoot_kernel kernel, const double* warp_a,
                  const double* warp_b, double c, bool learn_warp, std::vector<double>& Xu, std::vector<double>& r) {
  if (learn_warp && (warp_a || warp_b))
    return fail(SCOOT_ERR_INVALID_ARG, "gp nll: a learned warp takes no fixed warp_a / warp_b");
  return mle_inputs(X, y, m, d, kernel, warp_a, warp_b, c, learn_warp, Xu, r);
}

}  // namespace

int mle_nll_device(const double* X, const double* y, int m, int d, scoot_kernel kernel, const double* warp_a,
                   const double* warp_b, double c, bool learn_warp, const double* theta, double* nll, double* grad,
                   void* stream) {
  if (!theta || !nll) return fail(SCOOT_ERR_INVALID_ARG, "gp nll: null pointer");
  std::vector<double> Xu, r;
  int rc = device_inputs(X, y, m, d, kernel, warp_a, warp_b, c, learn_warp, Xu, r);
  if (rc != SCOOT_OK) return rc;
  const int P = learn_warp ? 3 * d + 2 : d + 2;
  for (int k = 0; k < P; ++k)
    if (!std::isfinite(theta[k])) return fail(SCOOT_ERR_INVALID_ARG, "gp nll: non-finite theta");
  DeviceNll dev;
  rc = dev.init(Xu, r, m, d, kernel, learn_warp, (hipStream_t)stream);
  if (rc != SCOOT_OK) return rc;
  const bool ok = dev.eval(theta, nll, grad);
  if (dev.error() != SCOOT_OK) return dev.error();
  if (!ok) return fail(SCOOT_ERR_NOT_PD, "gp nll: K is not positive definite");
  return SCOOT_OK;
}

int mle_fit_device(const double* X, const double* y, int m, int d, scoot_kernel kernel, const double* warp_a,
                   const double* warp_b, double c, bool learn_warp, const double* lower, const double* upper,
                   int max_iter, double* theta, double* nll_out, int* iters_out, void* stream) {
  std::vector<double> Xu, r;
  int rc = device_inputs(X, y, m, d, kernel, warp_a, warp_b, c, learn_warp, Xu, r);
  if (rc != SCOOT_OK) return rc;
  DeviceNll dev;
  rc = dev.init(Xu, r, m, d, kernel, learn_warp, (hipStream_t)stream);
  if (rc != SCOOT_OK) return rc;
  rc = lbfgs_box([&](const double* t, double* f, double* g) { return dev.eval(t, f, g); },
                 learn_warp ? 3 * d + 2 : d + 2, lower, upper, max_iter, theta, nll_out, iters_out);
  if (dev.error() != SCOOT_OK) return dev.error();
  return rc;
}

namespace {
// The GP at theta from a factorization on dev: the host part of a fit, with
// L^-1 and alpha from the device.
int gp_from_device(DeviceNll& dev, const double* X, const double* y, int m, int d, scoot_kernel kernel,
                   const double* warp_a, const double* warp_b, double c, bool learn_warp, const double* theta,
                   scoot_dtype dt, scoot_gp* out) {
  double ls[SCOOT_MAX_DIM], wa[SCOOT_MAX_DIM], wb[SCOOT_MAX_DIM];
  for (int k = 0; k < d; ++k) ls[k] = std::exp(theta[k]);
  const double* pa = warp_a;
  const double* pb = warp_b;
  if (learn_warp) {
    for (int k = 0; k < d; ++k) {
      wa[k] = std::exp(theta[d + 2 + k]);
      wb[k] = std::exp(theta[2 * d + 2 + k]);
    }
    pa = wa;
    pb = wb;
  }
  FitHost f;
  int rc = fit_setup(X, y, m, d, kernel, ls, pa, pb, std::exp(theta[d]), std::exp(theta[d + 1]), c, f);
  if (rc != SCOOT_OK) return rc;
  auto failed = [&]() {
    return dev.error() != SCOOT_OK ? dev.error()
                                   : fail(SCOOT_ERR_NOT_PD, "gp fit: K + tau^2 I is not positive definite");
  };
  if (dt == SCOOT_F32) {
    // fp32: packed on the device; the factorization's status is read after the
    // one synchronisation, and a handle made from a failed one is dropped
    if (!dev.launch_factor(theta)) return failed();
    scoot_gp gp = nullptr;
    rc = gp_from_factor(f, pa, pb, dev.Xi(), dev.blocks(), dev.alpha(), dev.stream(), &gp);
    if (rc != SCOOT_OK) return rc;
    if (!dev.factored()) {
      scoot_gp_destroy(gp);
      return failed();
    }
    *out = gp;
    return SCOOT_OK;
  }
  if (!dev.inverse(theta, f.Linv, f.alpha)) return failed();
  return gp_from_fit(f, pa, pb, dt, out);
}
}  // namespace

int mle_fit_device_gp(const double* X, const double* y, int m, int d, scoot_kernel kernel, const double* warp_a,
                      const double* warp_b, double c, bool learn_warp, const double* lower, const double* upper,
                      int max_iter, double* theta, scoot_dtype dt, void* stream, scoot_gp* out) {
  std::vector<double> Xu, r;
  int rc = device_inputs(X, y, m, d, kernel, warp_a, warp_b, c, learn_warp, Xu, r);
  if (rc != SCOOT_OK) return rc;
  DeviceNll dev;
  rc = dev.init(Xu, r, m, d, kernel, learn_warp, (hipStream_t)stream);
  if (rc != SCOOT_OK) return rc;
  rc = lbfgs_box([&](const double* t, double* f, double* g) { return dev.eval(t, f, g); },
                 learn_warp ? 3 * d + 2 : d + 2, lower, upper, max_iter, theta, nullptr, nullptr);
  if (dev.error() != SCOOT_OK) return dev.error();
  if (rc != SCOOT_OK) return rc;
  return gp_from_device(dev, X, y, m, d, kernel, warp_a, warp_b, c, learn_warp, theta, dt, out);
}

int gp_fit_device(const double* X, const double* y, int m, int d, scoot_kernel kernel, const double* ls,
                  const double* warp_a, const double* warp_b, double s2, double tau2, double c, scoot_dtype dt,
                  void* stream, scoot_gp* out) {
  if (!ls) return fail(SCOOT_ERR_INVALID_ARG, "gp fit: null pointer");
  if (d < 1 || d > SCOOT_MAX_DIM) return fail(SCOOT_ERR_INVALID_ARG, "gp fit: bad d");
  for (int k = 0; k < d; ++k)
    if (!(ls[k] > 0) || !std::isfinite(ls[k]))
      return fail(SCOOT_ERR_INVALID_ARG, "gp fit: lengthscales must be finite and > 0");
  if (!(s2 > 0) || !std::isfinite(s2) || !(tau2 > 0) || !std::isfinite(tau2))
    return fail(SCOOT_ERR_INVALID_ARG, "gp fit (device): signal and noise variance must be finite and > 0");
  double theta[SCOOT_MAX_DIM + 2];
  for (int k = 0; k < d; ++k) theta[k] = std::log(ls[k]);
  theta[d] = std::log(s2);
  theta[d + 1] = std::log(tau2);
  std::vector<double> Xu, r;
  int rc = device_inputs(X, y, m, d, kernel, warp_a, warp_b, c, false, Xu, r);
  if (rc != SCOOT_OK) return rc;
  DeviceNll dev;
  rc = dev.init(Xu, r, m, d, kernel, false, (hipStream_t)stream);
  if (rc != SCOOT_OK) return rc;
  return gp_from_device(dev, X, y, m, d, kernel, warp_a, warp_b, c, false, theta, dt, out);
}

}  // namespace scoot

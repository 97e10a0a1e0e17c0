// GP posterior over a candidate pool (Sec. 4.3, Eq. 4-5), fused:
//
//   K*[c, i] = k(x_c, X_i)                     Matern-5/2 ARD, generated on chip
//   mu[c]    = c0 + sum_i K*[c, i] alpha_i      (Eq. 4)
//   V        = L^-1 K*^T                         triangular product on matrix cores
//   sigma[c] = sqrt(max(0, s2 - sum_i V[i, c]^2))   (Eq. 5, latent f)
//   ei[c]    = G(best + xi)   optional fused EI epilogue (Eq. 8)
//
// One workgroup owns a tile of candidates at a time.  K* is made on chip and
// goes into LDS in the B-operand order of the matrix instruction, alpha folded
// in on the way (mu); the waves share the row blocks of V and keep only the
// squared norms of their rows.  In fp32 the observation blocks are the outer loop
// and K* of the next one is made beside the product of this one; in fp64 a tile
// goes through generation, product and reduction in turn.  K* and V never touch
// HBM.  L^-1 is shared by every workgroup (L2-resident).
//
// Covariance with folded constants: with per-dimension scale
// w_k = sqrt5 * log2(e) / l_k, u = sqrt(sum_k (w_k (x_k - X_ik))^2) equals
// sqrt5 r log2(e), and k = (c0 + u (c1 + u c2)) 2^-u with c0 = s2,
// c1 = s2 ln2, c2 = s2 ln2^2 / 3.  Observations arrive pre-scaled; padding rows
// sit at coordinate 1e4 (fp64) or carry a squared norm of 1e30 (the fp32
// augmented rows), so their covariance underflows to exactly 0, and their
// alpha and L^-1 entries are 0.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstring>
#include <type_traits>
#include <utility>

#include "internal.h"
#include "normal.h"

namespace scoot {

typedef float f4_t __attribute__((ext_vector_type(4)));
typedef float f16_t __attribute__((ext_vector_type(16)));
typedef double d2_t __attribute__((ext_vector_type(2)));
typedef double d4_t __attribute__((ext_vector_type(4)));

// E[(c - Y)^+] for Y ~ N(mu, sd^2), in double (epilogue only).
__device__ inline double partial_expectation_d(double c, double mu, double sd) {
  if (!(sd > 0)) return fmax(c - mu, 0.0);
  return sd * h_normal((c - mu) / sd);
}

// ---------------------------------------------------------------------------
// fp32.  A workgroup of RS waves owns a tile of 64 candidates (32 in small
// pools); wave r owns the row blocks (32 rows) of V that fall to it, for all of
// them.
//
// Squared distances on the fp64 matrix cores: with augmented rows
// A_i = (2 X_i, -|X_i|^2, -1) for the observations and B_x = (x, 1, |x|^2)
// for the candidates (scaled coordinates, fp64), A_i . B_x = -|x - X_i|^2, so
// one v_mfma_f64_16x16x4f64 chain over S = ceil((d + 2) / 4) steps gives -u^2
// for 16 observations x 16 candidates, exact to double rounding (no
// cancellation that float could see).  The observations are packed so that
// lane l = 16g + c, register r holds observation 16j + 4g + r of candidate c
// (the instruction's own order is row g + 4r there); the lane turns its four
// values into K* in float (sqrt, exp2, the polynomial) and folds alpha into
// the mean.
//
// The product V = L^-1 K*^T runs on the bf16 matrix cores without giving up
// fp32: every float is exactly the sum of three bfloat16 (8 + 8 + 8 bits), so
// with L^-1 = a1 + a2 + a3 (split on the host, from double) and K* = b1 + b2 +
// b3 (split in registers) a product is the six terms a1 b1, a1 b2, a2 b1,
// a2 b2, a1 b3, a3 b1, accumulated in float, smallest first; the three terms
// left out are below 2^-25 of the product.  Error against 64 bits, 2-norm over
// the pool and root mean square over data sets, with fp32 MFMA chains and now:
// m = 32 (200 sets) mu 2.4e-7 and 2.2e-7, sigma 4.0e-8 and 3.6e-8; m = 256 (40)
// 3.7e-7 and 3.1e-7, 5.3e-8 and 4.7e-8; m = 512 (24) 4.8e-7 and 4.0e-7, 5.0e-8 and
// 4.3e-8: the instruction rounds a sum of 16 products once or twice, to
// nearest, the fp32 one after every product.  Why: six bf16 instructions take
// 6/16 of the fp32 instruction's time, and while the fp32 matrix instruction
// and the vector ALU exclude each other, a bf16 one leaves the vector ALU free
// for about 19 of its 32 cycles (measured), which the K* generation of this
// wave and of the others on its SIMD can use.
//
// Loop order: observation blocks j of 16 outermost, and inside the row blocks
// P >= j / 2, their accumulators (two 32 x 32 tiles of 16 registers each)
// resident for the whole tile.  Row block nb - 1 - s is slot s; wave r owns
// slots r, r + RS, ..., so that at every j the live slots are the first ones
// of every wave.  The waves share the generation: wave r makes K* of block
// j + 1 for 64 / RS of the candidates (tiles of 32: the two waves whose slots
// die first, for 16 each) while the product of block j runs, and
// the parts go through LDS in the order of the product's B operand (lane l:
// observations 8 (l / 32) .. + 7 of candidate l % 32), two buffers, one barrier
// per j.  Executed matrix work is (nb32 + 1) / nb32 of the triangle's.
//
// L^-1 comes straight from L2 into registers, in units (32 rows x 16 columns,
// three parts, 3 KiB), each slot's next unit requested as soon as the slot's
// matrix instructions of this j are issued.  A unit feeds twelve matrix
// instructions (384 cycles); at two waves per SIMD a CU reads about 20 bytes
// per cycle.
//
// Bound: issue.  Per 32 candidates at m = 256 a SIMD needs 13.8k cycles of bf16
// and 6.1k of fp64 matrix instructions and about 9k of vector instructions,
// and takes 34k: the phases overlap little (the fp64 instructions exclude the
// vector ALU, and two waves often want the same unit).  Against the kernel with
// fp32 MFMA: 183 -> 141 us at m = 256, 69 -> 43 at m = 128, 286 -> 195 at m =
// 300, 2559 -> 1700 at m = 512 and n = 2^20 (n = 262,144 otherwise).  A ring of
// L^-1 units in LDS (four waves of 32 candidates each, every wave with all row
// blocks) took 135 us at m = 256 but 52 at m = 128 and 2210 at m = 512, where
// one wave per SIMD is left; K* two blocks ahead instead of one: no faster.
// ---------------------------------------------------------------------------
struct Post32 {
  int64_t n;
  int nj, nb32;  // observation blocks of 16, row blocks of 32
  int d;
  double scale[SCOOT_MAX_DIM];
  float c0, c1, c2;  // K* is made divided by 4^s2_exp
  double s2, vscale, prior, ei_c;  // vscale = 4^s2_exp: a squared norm times it is part of the variance
};

constexpr int kUnitBytes = 3 * 64 * 16;   // a unit's three parts in A-operand order

typedef __bf16 bf2_t __attribute__((ext_vector_type(2)));
typedef __bf16 bf8_t __attribute__((ext_vector_type(8)));
typedef float f2_t __attribute__((ext_vector_type(2)));
typedef unsigned u2_t __attribute__((ext_vector_type(2)));
typedef unsigned u4_t __attribute__((ext_vector_type(4)));

// Two floats as packed bf16 (round to nearest even); the floats become the
// (exact) remainders, x - 1.0 * low and y - 1.0 * high by the two-term bf16
// dot product.  neg = {(-1, 0), (0, -1)} must come from registers: given as
// constants the compiler writes (-1, 0) as the inline operand -1.0, which the
// instruction reads as (0, -1) (seen in a comparison with the plain form).
struct NegPairs {
  unsigned lo = 0x0000bf80u, hi = 0xbf800000u;
  __device__ NegPairs() { asm volatile("" : "+s"(lo), "+s"(hi)); }
};
__device__ inline unsigned split_bf16(float& x, float& y, const NegPairs& neg) {
  const bf2_t p = __builtin_convertvector(f2_t{x, y}, bf2_t);
  x = __builtin_amdgcn_fdot2_f32_bf16(p, __builtin_bit_cast(bf2_t, neg.lo), x, false);
  y = __builtin_amdgcn_fdot2_f32_bf16(p, __builtin_bit_cast(bf2_t, neg.hi), y, false);
  return __builtin_bit_cast(unsigned, p);
}
__device__ inline unsigned pack_bf16(float x, float y) {
  return __builtin_bit_cast(unsigned, __builtin_convertvector(f2_t{x, y}, bf2_t));
}
__device__ inline void mfma_bf16(const u4_t& a, const u4_t& b, f16_t& c) {
  c = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf8_t, a), __builtin_bit_cast(bf8_t, b), c, 0, 0, 0);
}

// LDS of a workgroup: K* parts, the candidates' augmented rows, the next
// tile's coordinates, the reductions.
template <int S, int RS, int H>
struct PostLds {
  u4_t b[2][H][3][64];      // [buffer][32-candidate half][part][lane]
  double bq[2 * H][S][64];  // [16-candidate tile][step][lane]
  float xb[2 * H][S][64];
  double sq[RS][64], mu[64];
  double scale[S * 4];
};

// S: fp64 MFMA steps of the distances; RS: waves that share a tile's rows;
// NBW: slots per wave; KA: register sets for units of L^-1; WPS: waves per SIMD
// that the register budget is set for; H: halves of 32 candidates in a tile.
template <int S, int RS, int NBW, int KA, int WPS, int H>
__global__ __launch_bounds__(RS * 64, WPS) void posterior_f32_kernel(
    const float* __restrict__ Xc, const unsigned char* __restrict__ linv, const double* __restrict__ xq,
    const float* __restrict__ alpha, float* __restrict__ mu_out, float* __restrict__ sd_out,
    float* __restrict__ ei_out, const Post32 a) {
  static_assert(RS == 4 || (RS == 2 && H == 2), "a wave makes whole tiles of K*");
  constexpr int TILE = 32 * H;    // candidates per workgroup and tile
  constexpr int GW = RS < 2 * H ? RS : 2 * H;  // waves that make K*
  constexpr int CT = 2 * H / GW;  // 16-candidate tiles whose K* such a wave makes
  constexpr int NP = 2 * CT;      // pieces of that work, two observations each
  // A wave of one or two slots and one tile of 16 candidates to generate has
  // little to hide its chain of distances, values and splits behind: the
  // distances run before the product, and both pieces stand between the matrix
  // instructions of the first slot, the last to die, four vector instructions
  // after each.  Left to the compiler, the pieces follow the product (m = 128: n
  // = 16,000 9.3 -> 8.8 us, 48,000 16.3 -> 15.0; m = 256: 24,000 21.6 -> 20.0).
  constexpr bool EARLY = CT == 1 && NBW <= 2;
  constexpr int PPS = EARLY ? NP : (NP + NBW - 1) / NBW;  // pieces beside a slot, in order
  const NegPairs neg;
  __shared__ PostLds<S, RS, H> sm;
  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int g = lane >> 4, c = lane & 15;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  // Two workgroups of a CU own their slots in opposite orders, since the first
  // slots live longest (workgroups gridDim / 2 apart usually share a CU).
  const int r = blockIdx.x >= (gridDim.x + 1) / 2 ? RS - 1 - wave : wave;
  const int64_t n_tiles = (a.n + TILE - 1) / TILE;
  // K* is made by every wave, or by those whose slots are the first to die
  const int gi = GW == RS ? wave : r - (RS - GW);
  const bool gen = GW == RS || gi >= 0;

  if (tid < S * 4) sm.scale[tid] = tid < a.d ? a.scale[min(tid, SCOOT_MAX_DIM - 1)] : 0.0;
  __syncthreads();

  // ---- this wave's 16-candidate tiles: coordinates and augmented rows -------
  // step s of the distance chain reads component k = 4s + g
  float xr[CT][S];
  auto load_x = [&](int64_t t) {
#pragma unroll
    for (int q = 0; q < CT; ++q) {
      const int64_t cand = min(t * TILE + (gi * CT + q) * 16 + c, a.n - 1);
#pragma unroll
      for (int s = 0; s < S; ++s) xr[q][s] = Xc[cand * a.d + min(4 * s + g, a.d - 1)];
    }
  };
  auto store_x = [&]() {
#pragma unroll
    for (int q = 0; q < CT; ++q)
#pragma unroll
      for (int s = 0; s < S; ++s) sm.xb[gi * CT + q][s][lane] = xr[q][s];
  };
  auto operands = [&]() {
#pragma unroll
    for (int q = 0; q < CT; ++q) {
      double x[S], nrm = 0.0;
#pragma unroll
      for (int s = 0; s < S; ++s) {
        x[s] = (double)sm.xb[gi * CT + q][s][lane] * sm.scale[4 * s + g];
        if (4 * s + g < a.d) nrm = fma(x[s], x[s], nrm);
      }
      nrm += __shfl_xor(nrm, 16);
      nrm += __shfl_xor(nrm, 32);
#pragma unroll
      for (int s = 0; s < S; ++s) {
        const int k = 4 * s + g;
        sm.bq[gi * CT + q][s][lane] = k < a.d ? x[s] : (k == a.d ? 1.0 : (k == a.d + 1 ? nrm : 0.0));
      }
    }
  };

  // ---- K* of an observation block, in pieces ---------------------------------
  // Piece 2q makes the distances of tile q and its first two observations'
  // values, piece 2q + 1 the other two and the LDS writes.
  double aq[S];
  f4_t al;
  auto load_obs = [&](int j) {
#pragma unroll
    for (int s = 0; s < S; ++s) aq[s] = (xq + (size_t)j * S * 64)[(unsigned)(s * 64 + lane)];
    al = reinterpret_cast<const f4_t*>(alpha + 16 * j)[(unsigned)g];
  };
  double mu_acc[CT];
#pragma unroll
  for (int q = 0; q < CT; ++q) mu_acc[q] = 0.0;
  d4_t cr;
  float m_part;
  unsigned pk[3][2];
  auto distances = [&](int q) {
    cr = d4_t{0.0, 0.0, 0.0, 0.0};
#pragma unroll
    for (int s = 0; s < S; ++s)
      cr = __builtin_amdgcn_mfma_f64_16x16x4f64(aq[s], sm.bq[gi * CT + q][s][lane], cr, 0, 0, 0);
  };
  auto piece = [&](int p, int to_buf) {
    const int q = p >> 1, h = p & 1;
    if (h == 0) {
      if constexpr (!EARLY) distances(q);
      m_part = 0.0f;
    }
    float kv[2];
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      const float u = __builtin_amdgcn_sqrtf(fmaxf((float)(-cr[2 * h + i]), 0.0f));
      kv[i] = fmaf(u, fmaf(u, a.c2, a.c1), a.c0) * __builtin_amdgcn_exp2f(-u);
      m_part = fmaf(kv[i], al[2 * h + i], m_part);
    }
    pk[0][h] = split_bf16(kv[0], kv[1], neg);
    pk[1][h] = split_bf16(kv[0], kv[1], neg);
    pk[2][h] = pack_bf16(kv[0], kv[1]);
    if (h == 1) {
      mu_acc[q] += (double)m_part;
      const int ct = gi * CT + q;
      u4_t* to = &sm.b[to_buf][ct >> 1][0][(g >> 1) * 32 + (ct & 1) * 16 + c];
#pragma unroll
      for (int part = 0; part < 3; ++part)
        reinterpret_cast<u2_t*>(to + part * 64)[g & 1] = u2_t{pk[part][0], pk[part][1]};
    }
  };

  // ---- L^-1 ----------------------------------------------------------------
  // Register set k holds the units of slots k, k + KA, ... one after the other,
  // and then block j + 1's of slot k (the next tile's block 0 once that slot
  // has died).  Every index is within the stream.
  u4_t au[KA][3];
  auto load_unit = [&](int k, int unit) {
    const u4_t* at = reinterpret_cast<const u4_t*>(linv + (size_t)unit * kUnitBytes);
#pragma unroll
    for (int part = 0; part < 3; ++part) au[k][part] = at[(unsigned)(part * 64 + lane)];
  };
  auto first_unit = [&](int k) { return min(r + RS * k, a.nb32 - 1); };

  int64_t tile = blockIdx.x;
  if (gen) {
    load_x(tile);
    store_x();
    load_obs(0);
  }
#pragma unroll
  for (int k = 0; k < KA; ++k) load_unit(k, first_unit(k));
  if (gen) {
    operands();
    if constexpr (EARLY) distances(0);
#pragma unroll
    for (int p = 0; p < NP; ++p) piece(p, 0);
    load_obs(a.nj > 1 ? 1 : 0);
    load_x(tile + gridDim.x);
    store_x();
  }
  int buf = 0;  // the buffer that holds K* of the block being multiplied
  f16_t acc[NBW][H];

  for (; tile < n_tiles; tile += gridDim.x) {
    const int64_t c0 = tile * TILE;
#pragma unroll
    for (int t = 0; t < NBW; ++t)
#pragma unroll
      for (int h = 0; h < H; ++h)
#pragma unroll
        for (int i = 0; i < 16; ++i) acc[t][h][i] = 0.0f;

    int off = 0;  // first unit of block j
#pragma unroll 1
    for (int j = 0; j < a.nj; ++j) {
      const int live = a.nb32 - (j >> 1);
      __syncthreads();  // K* of block j is in LDS
      u4_t bc[H][3];
#pragma unroll
      for (int part = 0; part < 3; ++part)
#pragma unroll
        for (int h = 0; h < H; ++h) bc[h][part] = sm.b[buf][h][part][lane];
      buf ^= 1;
      // block to generate beside this product, and the one after it
      int jn = j + 1;
      const int cur = off;
      off += live;
      int noff = off, nlive = a.nb32 - (jn >> 1);
      if (jn == a.nj) {
        // every K* of this tile is made: its mean is complete, and the next
        // tile's first block is generated beside this tile's last rows
#pragma unroll
        for (int q = 0; q < CT; ++q) {
          mu_acc[q] += __shfl_xor(mu_acc[q], 16);
          mu_acc[q] += __shfl_xor(mu_acc[q], 32);
          if (gen && g == 0) sm.mu[(gi * CT + q) * 16 + c] = mu_acc[q];
          mu_acc[q] = 0.0;
        }
        if (gen) operands();
        jn = 0;
        noff = 0;
        nlive = a.nb32;
      }
      if constexpr (EARLY)
        if (gen) distances(0);
#pragma unroll
      for (int t = 0; t < NBW; ++t) {
        if (r + RS * t < live) {
          // the matrix phases go first: the other waves' vector work fills the
          // gaps between their instructions (3-4% per launch)
          __builtin_amdgcn_s_setprio(2);
#pragma unroll
          for (int h = 0; h < H; ++h) mfma_bf16(au[t % KA][2], bc[h][0], acc[t][h]);
#pragma unroll
          for (int h = 0; h < H; ++h) mfma_bf16(au[t % KA][0], bc[h][2], acc[t][h]);
#pragma unroll
          for (int h = 0; h < H; ++h) mfma_bf16(au[t % KA][1], bc[h][1], acc[t][h]);
#pragma unroll
          for (int h = 0; h < H; ++h) mfma_bf16(au[t % KA][1], bc[h][0], acc[t][h]);
#pragma unroll
          for (int h = 0; h < H; ++h) mfma_bf16(au[t % KA][0], bc[h][1], acc[t][h]);
#pragma unroll
          for (int h = 0; h < H; ++h) mfma_bf16(au[t % KA][0], bc[h][0], acc[t][h]);
          {
            const int k = t % KA, sn = r + RS * k;  // the set, and its first slot
            int unit = sn < nlive ? noff + sn : first_unit(k);
            if (t + KA < NBW && r + RS * (t + KA) < live) unit = cur + r + RS * (t + KA);
            load_unit(k, unit);
          }
          if (gen) {
#pragma unroll
            for (int p = t * PPS; p < NP && p < (t + 1) * PPS; ++p) piece(p, buf);
          }
          if (EARLY && t == 0) {
#pragma unroll
            for (int i = 0; i < 6 * H; ++i) {
              __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);  // a matrix instruction
              __builtin_amdgcn_sched_group_barrier(0x002, 4, 0);  // and four vector ones
            }
          }
          __builtin_amdgcn_s_setprio(0);
          asm volatile("; slot %0" ::"i"(t));  // keeps the two copies of the pieces apart
        } else if (gen) {
#pragma unroll
          for (int p = t * PPS; p < NP && p < (t + 1) * PPS; ++p) piece(p, buf);
        }
      }
      if (gen) load_obs(jn + 1 < a.nj ? jn + 1 : 0);
    }
    // ---- squared norms of the columns -----------------------------------------
    if (gen) load_x(tile + 2 * (int64_t)gridDim.x);
#pragma unroll
    for (int h = 0; h < H; ++h) {
      double sq = 0.0;
#pragma unroll
      for (int t = 0; t < NBW; ++t) {
        if (r + RS * t < a.nb32) {
          float q[4] = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
          for (int i = 0; i < 16; ++i) q[i & 3] = fmaf(acc[t][h][i], acc[t][h][i], q[i & 3]);
          sq += (double)((q[0] + q[1]) + (q[2] + q[3]));
        }
      }
      sq += __shfl_xor(sq, 32);
      if (lane < 32) sm.sq[wave][h * 32 + lane] = sq;
    }
    if (gen) store_x();
    __syncthreads();
    const int64_t cand = c0 + lane;
    if (wave == 0 && lane < TILE && cand < a.n) {
      double sq = 0.0;
#pragma unroll
      for (int w = 0; w < RS; ++w) sq += sm.sq[w][lane];
      const double sd = sqrt(fmax(a.s2 - a.vscale * sq, 0.0));
      const double mu = a.prior + sm.mu[lane];
      mu_out[cand] = (float)mu;
      sd_out[cand] = (float)sd;
    }
  }
  // The EI of the candidates whose mean and deviation this lane has written;
  // in a loop of its own, so that the constants of the tail and exp hold no
  // registers beside the accumulators.
  if (ei_out && wave == 0) {
    for (tile = blockIdx.x; tile < n_tiles; tile += gridDim.x) {
      const int64_t cand = tile * TILE + lane;
      if (lane < TILE && cand < a.n) ei_out[cand] = (float)partial_expectation_d(a.ei_c, (double)mu_out[cand], (double)sd_out[cand]);
    }
  }
}

// ---------------------------------------------------------------------------
// fp64: v_mfma_f64_16x16x4f64 on 16 x 16 blocks, tiles of 32 candidates (two
// 16-column MFMA tiles ct = 0, 1).  At MFMA step s (0..3) of block (I, J), A
// lane l holds Linv[16I + l%16][16J + 4s + l/16] and B lane l holds
// K*[16J + 4s + l/16][16ct + l%16]; K* is stored as (J, ct, s/2, lane)
// double2, component s%2.  Accumulator register r of lane l holds row
// l/16 + 4r, column l%16 of its tile (only column sums of squares are taken,
// so the row order does not matter here).  A persistent workgroup takes every
// tile through three phases:
//   1. generate: every wave computes K* for a share of the observation rows, for
//      all candidates of the tile;
//   2. multiply: every wave takes whole row blocks I of V (a per-SIMD row plan
//      keeps the triangular work balanced), sum_{J<=I} Linv[I,J] K*[J] with A
//      from the packed L^-1 in L2 and B from LDS;
//   3. reduce: partial norms and means of all waves are summed per candidate.
// ---------------------------------------------------------------------------
struct Post64 {
  int64_t n;
  int d, nb16;
  double scale[SCOOT_MAX_DIM];
  double c0, c1, c2;
  double s2, prior, ei_c;
  int warp;  // candidates through kumaraswamy(x, wa, wb) first
  double wa[SCOOT_MAX_DIM], wb[SCOOT_MAX_DIM];
  RowPlan16 plan;  // 16-row blocks
};

__device__ inline void load_block16(d2_t (&a)[2], const d2_t* ap, int k) {
  a[0] = ap[(size_t)(k * 2 + 0) * 64];
  a[1] = ap[(size_t)(k * 2 + 1) * 64];
}
// b[2 ct + s/2]
__device__ inline void load_b16(d2_t (&b)[4], const d2_t* ks, int J, int lane) {
#pragma unroll
  for (int ct = 0; ct < 2; ++ct)
#pragma unroll
    for (int s2 = 0; s2 < 2; ++s2) b[2 * ct + s2] = ks[((J * 2 + ct) * 2 + s2) * 64 + lane];
}

// The 4 steps of a block on two chains (one per 16-candidate half), issued
// alternately; FIRST (the row's block J = 0) starts both from zero, so they need no
// clearing.
template <bool FIRST>
__device__ inline void mfma_block16(d4_t& l0, d4_t& l1, const d2_t (&a)[2], const d2_t (&b)[4]) {
  const d4_t zero = {0};
#pragma unroll
  for (int s2 = 0; s2 < 2; ++s2) {
#pragma unroll
    for (int t = 0; t < 2; ++t) {
      const bool z = FIRST && s2 == 0 && t == 0;
      l0 = __builtin_amdgcn_mfma_f64_16x16x4f64(a[s2][t], b[s2][t], z ? zero : l0, 0, 0, 0);
      l1 = __builtin_amdgcn_mfma_f64_16x16x4f64(a[s2][t], b[2 + s2][t], z ? zero : l1, 0, 0, 0);
    }
  }
}
__device__ inline void mfma_block16_at(int J, d4_t& l0, d4_t& l1, const d2_t (&a)[2], const d2_t (&b)[4]) {
  if (J == 0) mfma_block16<true>(l0, l1, a, b);
  else mfma_block16<false>(l0, l1, a, b);
}

// One tile's pass over the wave's blocks: one block of read-ahead, the A stream
// wrapping to the next tile.
__device__ inline void wave_tile16(const d2_t* __restrict__ ap, const d2_t* ks, uint64_t lo, uint64_t hi, int count,
                                   int lane, d2_t (&ax)[2], double& sq0, double& sq1) {
  d4_t l0 = __builtin_nondeterministic_value(l0), l1 = l0;
  constexpr uint64_t kMask = (1u << kRowBits16) - 1;
  int I = (int)(lo & kMask), J = 0;
  auto next_j = [&](int j, int i) { return j == i ? 0 : j + 1; };
  auto advance = [&]() {
    if (J == I) {
      double p0 = 0.0, p1 = 0.0;
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        p0 = fma(l0[r], l0[r], p0);
        p1 = fma(l1[r], l1[r], p1);
      }
      sq0 += p0;
      sq1 += p1;
      J = 0;
      lo = (lo >> kRowBits16) | (hi << (64 - kRowBits16));
      hi >>= kRowBits16;
      I = (int)(lo & kMask);
    } else {
      ++J;
    }
  };
  d2_t ay[2], bx[4], by[4];
  load_b16(bx, ks, 0, lane);
  int k = 0;
  for (; k + 1 < count; k += 2) {
    load_block16(ay, ap, k + 1);
    load_b16(by, ks, next_j(J, I), lane);
    __builtin_amdgcn_sched_barrier(0);
    mfma_block16_at(J, l0, l1, ax, bx);
    __builtin_amdgcn_sched_barrier(0);
    advance();
    load_block16(ax, ap, k + 2 < count ? k + 2 : 0);
    load_b16(bx, ks, next_j(J, I), lane);
    __builtin_amdgcn_sched_barrier(0);
    mfma_block16_at(J, l0, l1, ay, by);
    __builtin_amdgcn_sched_barrier(0);
    advance();
  }
  if (k < count) {
    load_block16(ay, ap, 0);
    __builtin_amdgcn_sched_barrier(0);
    mfma_block16_at(J, l0, l1, ax, bx);
    __builtin_amdgcn_sched_barrier(0);
    advance();
    ax[0] = ay[0];
    ax[1] = ay[1];
  }
}

template <int WAVES, int D>
__global__ __launch_bounds__(WAVES * 64, 8 / WAVES) void posterior_f64_kernel(
    const float* __restrict__ Xc, const d2_t* __restrict__ linv, const double* __restrict__ xs,
    const double* __restrict__ alpha, double* __restrict__ mu_out, double* __restrict__ sd_out,
    double* __restrict__ ei_out, const Post64 a) {
  extern __shared__ __align__(16) unsigned char smem[];
  d2_t* ks = reinterpret_cast<d2_t*>(smem);  // [nb16][2 ct][2 s2][64] double2
  const int nb = a.nb16;
  double* sig_red = reinterpret_cast<double*>(ks + (size_t)nb * 2 * 2 * 64);  // [WAVES][4 g][32]
  double* mu_red = sig_red + WAVES * 4 * 32;                                   // [WAVES][2 h][32]

  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int64_t n_tiles = (a.n + 31) >> 5;
  static_assert(WAVES % 2 == 0, "phase 1 relies on an even wave count");
  // 16-byte loads per observation row: the D coordinates and, below 16, alpha
  constexpr int kRowVec = D < kXsStride ? (D + 1 + 1) / 2 : kXsStride / 2;

  // Plan entry of this wave: of eight, the two of a SIMD take entries p and p + 4,
  // which the plan balances; by wave number if they did not land two to a SIMD.
  int p = wave;
  if constexpr (WAVES == 8) {
    int* on_simd = reinterpret_cast<int*>(mu_red + WAVES * 2 * 32);  // [4]
    if (tid < 4) on_simd[tid] = 0;
    __syncthreads();
    const int simd = (int)((__builtin_amdgcn_s_getreg((31 << 11) | 4) >> 4) & 3);  // HW_ID.SIMD_ID
    int slot = 0;
    if (lane == 0) slot = atomicAdd(&on_simd[simd], 1);
    slot = __shfl(slot, 0);
    __syncthreads();
    if (on_simd[0] == 2 && on_simd[1] == 2 && on_simd[2] == 2 && on_simd[3] == 2) p = simd + 4 * slot;
    p = __builtin_amdgcn_readfirstlane(p);
  }
  const uint64_t rows_lo = a.plan.lo[p], rows_hi = a.plan.hi[p];
  const int count = a.plan.blk_start[p + 1] - a.plan.blk_start[p];
  const d2_t* ap = linv + (size_t)a.plan.blk_start[p] * 2 * 64 + lane;
  d2_t ax[2];
  if (count > 0) load_block16(ax, ap, 0);

  // lane -> candidate 32 tile + cl, row half h
  const int cl = lane & 31, h = lane >> 5;
  const int ct = cl >> 4, ncol = cl & 15;
  int64_t tile = blockIdx.x;
  float xr[D];
#pragma unroll
  for (int q = 0; q < D; ++q) xr[q] = Xc[min(tile * 32 + cl, a.n - 1) * D + q];

  double last_mu = 0.0, last_sd = 0.0;  // of the newest tile
  for (; tile < n_tiles; tile += gridDim.x) {
    const int64_t c0 = tile * 32;
    double xc[D];
#pragma unroll
    for (int q = 0; q < D; ++q) {
      const double x = a.warp ? kumaraswamy((double)xr[q], a.wa[q], a.wb[q]) : (double)xr[q];
      xc[q] = x * a.scale[q];
    }
    const int64_t next = tile + gridDim.x;
    if (next < n_tiles) {
#pragma unroll
      for (int q = 0; q < D; ++q) xr[q] = Xc[min(next * 32 + cl, a.n - 1) * D + q];
    }

    __builtin_amdgcn_s_setprio(2);  // where a CU's waves are in different phases, generation is served first
    // ---- phase 1: group G = 4J + 2 s2 + kk covers rows
    // 16J + 8 s2 + 4t + 2kk + h = 4G - 2kk + h + 4t (t = 0, 1) of block J;
    // WAVES is even, so kk = wave & 1 for all of a wave's groups and each
    // lane's rows advance by 4 WAVES per group.
    double mu_part = 0.0;
    const int ngroups = nb * 4;
    const int kw = wave & 1;
    const double* xg = xs + (size_t)(4 * wave - 2 * kw + h) * kXsStride;
    for (int G = wave; G < ngroups; G += WAVES, xg += 4 * WAVES * kXsStride) {
      const int J = G >> 2, s2 = (G >> 1) & 1;
      d2_t kv;
#pragma unroll
      for (int t = 0; t < 2; ++t) {
        const double* xo = xg + 4 * t * kXsStride;
        double xv[kRowVec * 2];
#pragma unroll
        for (int r = 0; r < kRowVec; ++r) {
          const d2_t v2 = reinterpret_cast<const d2_t*>(xo)[r];
          xv[2 * r] = v2[0];
          xv[2 * r + 1] = v2[1];
        }
        double acc = 0.0;
#pragma unroll
        for (int q = 0; q < D; ++q) {
          const double df = xc[q] - xv[q];
          acc = fma(df, df, acc);
        }
        const double u = sqrt(acc);
        const double kval = fma(u, fma(u, a.c2, a.c1), a.c0) * exp2(-u);
        kv[t] = kval;
        const double al = D < kXsStride ? xv[D < kXsStride ? D : 0] : alpha[4 * G - 2 * kw + h + 4 * t];
        mu_part = fma(kval, al, mu_part);
      }
      ks[((J * 2 + ct) * 2 + s2) * 64 + (2 * kw + h) * 16 + ncol] = kv;
    }
    __syncthreads();

    __builtin_amdgcn_s_setprio(0);
    // ---- phase 2 ----------------------------------------------------------
    double sq0 = 0.0, sq1 = 0.0;
    if (count > 0) wave_tile16(ap, ks, rows_lo, rows_hi, count, lane, ax, sq0, sq1);

    // ---- phase 3: accumulator lane l holds column l % 16 of its tile ------
    const int g = lane >> 4;
    sig_red[(wave * 4 + g) * 32 + (lane & 15)] = sq0;
    sig_red[(wave * 4 + g) * 32 + 16 + (lane & 15)] = sq1;
    mu_red[(wave * 2 + h) * 32 + cl] = mu_part;
    __syncthreads();
    if (tid < 32) {
      const int64_t c = c0 + tid;
      if (c < a.n) {
        double ss = 0.0, mm = 0.0;
#pragma unroll
        for (int w = 0; w < WAVES; ++w) {
#pragma unroll
          for (int gg = 0; gg < 4; ++gg) ss += sig_red[(w * 4 + gg) * 32 + tid];
          mm += mu_red[(w * 2 + 0) * 32 + tid] + mu_red[(w * 2 + 1) * 32 + tid];
        }
        last_sd = sqrt(fmax(a.s2 - ss, 0.0));
        last_mu = a.prior + mm;
        mu_out[c] = last_mu;
        sd_out[c] = last_sd;
      }
    }
  }
  // The EI of the workgroup's candidates, after the loop as above: inside it the
  // tail's constants took 25 registers, and a third of the waves (a pass of one
  // objective, m = 32, n = 262,144 71 -> 85 us).  The last tile's from registers,
  // where small pools end.
  if (ei_out) {
    tile -= gridDim.x;
    if (tid < 32 && tile * 32 + tid < a.n) ei_out[tile * 32 + tid] = partial_expectation_d(a.ei_c, last_mu, last_sd);
    if (tile > blockIdx.x) {
      __syncthreads();  // the other tiles' means and deviations are written
      for (int64_t i = tid; blockIdx.x + (i >> 5) * gridDim.x < tile; i += WAVES * 64) {
        const int64_t c = (blockIdx.x + (i >> 5) * gridDim.x) * 32 + (i & 31);
        ei_out[c] = partial_expectation_d(a.ei_c, mu_out[c], sd_out[c]);
      }
    }
  }
}

// ---------------------------------------------------------------------------
// Packing of a device factorization for the fp32 kernel, as pack_linv_f32 does
// on the host: one wave per unit, eight entries (64 contiguous bytes of a
// factor block) per lane.  It replaces the read-back of L^-1, the host packing
// and the upload (m = 300: 0.7 MiB down and 0.33 MiB up).
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(64) void pack_f32_kernel(const double* __restrict__ Xi, int nbf,
                                                      const double* __restrict__ alpha, int m, int nb32, double lscale,
                                                      u4_t* __restrict__ linv, double* __restrict__ alpha64,
                                                      float* __restrict__ alpha32) {
  const int j = blockIdx.x, P = blockIdx.y, lane = threadIdx.x;
  if (j == 0 && P == 0) {
    for (int i = lane; i < nb32 * 32; i += 64) {
      const double v = i < m ? alpha[i] : 0.0;
      alpha64[i] = v;
      alpha32[i] = (float)(v * lscale * lscale);
    }
  }
  if (P < j / 2) return;
  // the units before block j's, then row blocks from the last one down
  const int unit = j * nb32 - (j - 1) * (j - 1) / 4 + nb32 - 1 - P;
  const int row = 32 * P + (lane & 31), col = 16 * j + 8 * (lane >> 5);
  u4_t part[3];
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    double v[2];
#pragma unroll
    for (int q = 0; q < 2; ++q) {
      const int c = col + 2 * i + q;
      const double* blk = Xi + ((size_t)(row >> 4) * nbf + (c >> 4)) * 256;
      v[q] = row < m && c <= row ? lscale * blk[(row & 15) * 16 + (c & 15)] : 0.0;
    }
#pragma unroll
    for (int p = 0; p < 3; ++p) {
      const unsigned w = pack_bf16((float)v[0], (float)v[1]);
      part[p][i] = w;
      v[0] -= (double)__builtin_bit_cast(float, w << 16);
      v[1] -= (double)__builtin_bit_cast(float, w & 0xffff0000u);
    }
  }
#pragma unroll
  for (int p = 0; p < 3; ++p) linv[((size_t)unit * 3 + p) * 64 + lane] = part[p];
}

int launch_pack_f32(const double* Xi, int nbf, const double* alpha, int m, int nb32, int s2_exp, void* linv,
                    double* alpha64, float* alpha32, void* stream) {
  hipLaunchKernelGGL(pack_f32_kernel, dim3((unsigned)((m + 15) / 16), (unsigned)nb32), dim3(64), 0,
                     (hipStream_t)stream, Xi, nbf, alpha, m, nb32, std::ldexp(1.0, s2_exp), (u4_t*)linv, alpha64,
                     alpha32);
  const hipError_t err = hipGetLastError();
  if (err != hipSuccess) return fail(SCOOT_ERR_DEVICE, std::string("gp fit: pack launch: ") + hipGetErrorString(err));
  return SCOOT_OK;
}

// ---------------------------------------------------------------------------
// Input warping of the pool (fp32 path): every coordinate through
// w = 1 - (1 - x^a_k)^b_k, x clamped to [0, 1], in float and without
// cancellation: ln x from log1p(x - 1) above 1/2 (x - 1 exact there),
// 1 - x^a = -expm1(a ln x), w = -expm1(b ln(1 - x^a)).  Measured against
// double: 2e-7 absolute (forming x^a first and subtracting it from 1 loses
// up to 1.5e-4 near x = 1, where w is steep).  The fp64 path warps in double
// inside its kernel, by the same steps.
// ---------------------------------------------------------------------------
struct WarpArgs {
  float a[SCOOT_MAX_DIM], b[SCOOT_MAX_DIM];
};

__global__ __launch_bounds__(256) void warp_pool_kernel(const float* __restrict__ Xc, int64_t total, int d,
                                                        const WarpArgs w, float* __restrict__ out) {
  for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < total; i += (int64_t)gridDim.x * 256) {
    const int k = (int)(i % d);
    const float x = fminf(fmaxf(Xc[i], 0.0f), 1.0f);
    const float lx = x > 0.5f ? log1pf(x - 1.0f) : logf(x);
    const float om = -expm1f(w.a[k] * lx);
    out[i] = -expm1f(w.b[k] * logf(om));
  }
}

int launch_warp_pool(const GPDevice& g, const float* Xc, int64_t n, float* out, void* stream) {
  const int64_t total = n * g.d;
  if (total == 0) return SCOOT_OK;
  WarpArgs w{};
  for (int k = 0; k < SCOOT_MAX_DIM; ++k) {
    w.a[k] = (float)g.warp_a[k];
    w.b[k] = (float)g.warp_b[k];
  }
  const int64_t blocks = std::min<int64_t>((total + 255) / 256, 8192);
  hipLaunchKernelGGL(warp_pool_kernel, dim3((unsigned)blocks), dim3(256), 0, (hipStream_t)stream, Xc, total, g.d,
                     w, out);
  hipError_t err = hipGetLastError();
  if (err != hipSuccess) return fail(SCOOT_ERR_DEVICE, std::string("warp launch: ") + hipGetErrorString(err));
  return SCOOT_OK;
}

// ---------------------------------------------------------------------------
// launchers
// ---------------------------------------------------------------------------
namespace {

// Persistent grid: as many workgroups as the chip holds at once (each loops
// over tiles), at most one per tile.  0 when the workgroup does not fit.
int64_t persistent_grid(const void* kern, int threads, size_t lds, int64_t tiles) {
  int dev = 0, cus = 256, per_cu = 0;
  (void)hipGetDevice(&dev);
  (void)hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev);
  if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, kern, threads, lds) != hipSuccess || per_cu < 1)
    return 0;
  return std::min(tiles, (int64_t)cus * per_cu);
}

template <int S, int RS, int NBW, int KA, int WPS, int H>
int run32(const GPDevice& g, const float* Xc, int64_t n, float* mu, float* sd, float* ei, const Post32& a,
          hipStream_t s) {
  auto kern = posterior_f32_kernel<S, RS, NBW, KA, WPS, H>;
  const int64_t grid = persistent_grid((const void*)kern, RS * 64, 0, (n + 32 * H - 1) / (32 * H));
  if (grid < 1) return fail(SCOOT_ERR_DEVICE, "posterior: workgroup does not fit on a compute unit");
  hipLaunchKernelGGL(kern, dim3((unsigned)grid), dim3(RS * 64), 0, s, Xc, (const unsigned char*)g.linv,
                     (const double*)g.xs, g.alpha32, mu, sd, ei, a);
  return SCOOT_OK;
}
template <int S>
int run32_by_rows(const GPDevice& g, const float* Xc, int64_t n, float* mu, float* sd, float* ei, const Post32& a,
                  hipStream_t s) {
  // Two waves share a tile where the pool fills the chip, four where it does
  // not: a tile alone takes them half the time, m = 128, n = 3000 12.1 -> 7.9
  // us, m = 224 20.0 -> 13.0.  The line: two-wave workgroups come four to a CU
  // (six up to m = 128), and four waves are the faster ones up to about three
  // tiles per CU (n = 48,000, m = 256 35.7 -> 30.3, but 64,000 38.6 -> 40.1), and
  // at m <= 128 up to the start of the second round of six (n = 100,000, m = 128
  // 31.0 -> 27.4, but 262,144 54.5 -> 58.1).  Tiles of 32 candidates, whose
  // blocks take half the matrix time, as long as every one has a CU to itself (n =
  // 8192: m = 64 6.4 -> 5.9, 128 8.7 -> 8.1, 192 12.2 -> 11.0, 256 15.2 -> 13.8);
  // two on a CU read L^-1 twice and are slower than one of 64 (n = 12,000, m =
  // 128 8.9 -> 10.0).  Registers for three waves per SIMD with two slots: n =
  // 48,000, m = 256 31.0 -> 28.4, at d = 16 (five distance steps) they spill: n =
  // 24,000 22.4 -> 24.4.
  int dev = 0, cus = 256;
  (void)hipGetDevice(&dev);
  (void)hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev);
  const int64_t tiles = (n + 63) / 64;
  constexpr int WPS = S <= 4 ? 3 : 2;
  const bool halves = (n + 31) / 32 <= cus;
  if (a.nb32 <= 4 && halves) return run32<S, 4, 1, 1, 2, 1>(g, Xc, n, mu, sd, ei, a, s);
  if (a.nb32 <= 8 && halves) return run32<S, 4, 2, 2, 2, 1>(g, Xc, n, mu, sd, ei, a, s);
  if (a.nb32 <= 4 && tiles <= 7 * (int64_t)cus) return run32<S, 4, 1, 1, 2, 2>(g, Xc, n, mu, sd, ei, a, s);
  if (a.nb32 <= 8 && tiles <= 3 * (int64_t)cus) return run32<S, 4, 2, 2, WPS, 2>(g, Xc, n, mu, sd, ei, a, s);
  if (a.nb32 <= 4) return run32<S, 2, 2, 2, 3, 2>(g, Xc, n, mu, sd, ei, a, s);
  if (a.nb32 <= 8) return run32<S, 2, 4, 3, 2, 2>(g, Xc, n, mu, sd, ei, a, s);
  if (a.nb32 <= 16) return run32<S, 4, 4, 4, 2, 2>(g, Xc, n, mu, sd, ei, a, s);
  return run32<S, 4, 5, 2, 2, 2>(g, Xc, n, mu, sd, ei, a, s);
}

template <int WAVES, int D>
int run64(const GPDevice& g, const float* Xc, int64_t n, double* mu, double* sd, double* ei,
          const Post64& a, hipStream_t s) {
  // K* tile, per-wave partial norms and means, four SIMD counters
  const int nb16 = g.m_pad / kBlk16;
  const size_t lds = (size_t)nb16 * 2 * 2 * 64 * 16 + WAVES * 4 * 32 * 8 + WAVES * 2 * 32 * 8 + 16;
  auto kern = posterior_f64_kernel<WAVES, D>;
  const int rc = allow_full_lds((const void*)kern, "posterior");
  if (rc != SCOOT_OK) return rc;
  const int64_t grid = persistent_grid((const void*)kern, WAVES * 64, lds, (n + 31) / 32);
  if (grid < 1) return fail(SCOOT_ERR_DEVICE, "posterior: workgroup does not fit on a compute unit");
  hipLaunchKernelGGL(kern, dim3((unsigned)grid), dim3(WAVES * 64), lds, s, Xc,
                     (const d2_t*)g.linv, (const double*)g.xs, g.alpha, mu, sd, ei, a);
  return SCOOT_OK;
}

template <int D, typename F>
int by_d_rec(int d, F&& f) {
  if constexpr (D > SCOOT_MAX_DIM) {
    return fail(SCOOT_ERR_UNSUPPORTED, "posterior: d exceeds SCOOT_MAX_DIM");
  } else {
    if (d == D) return f(std::integral_constant<int, D>());
    return by_d_rec<D + 1>(d, std::forward<F>(f));
  }
}

}  // namespace

int launch_posterior(const GPDevice& g, const float* Xc, int64_t n, void* mu, void* sigma,
                     const double* ei_c, void* ei, void* stream, bool xc_warped) {
  if (n == 0) return SCOOT_OK;
  if (n >= ((int64_t)1 << 37)) return fail(SCOOT_ERR_UNSUPPORTED, "posterior: n too large");
  hipStream_t s = (hipStream_t)stream;
  int rc;
  if (g.dt == SCOOT_F32 && g.warp && !xc_warped) {
    float* Xw = (float*)device_scratch((size_t)n * g.d * sizeof(float), 5);
    if (!Xw) return fail(SCOOT_ERR_NO_MEMORY, "posterior: warped pool allocation failed");
    rc = launch_warp_pool(g, Xc, n, Xw, stream);
    if (rc != SCOOT_OK) return rc;
    Xc = Xw;
  }
  if (g.dt == SCOOT_F32) {
    Post32 a{};
    a.n = n;
    a.d = g.d;
    a.nj = (g.m + 15) / 16;
    a.nb32 = g.nb;
    for (int k = 0; k < SCOOT_MAX_DIM; ++k) a.scale[k] = g.scale64[k];
    a.c0 = g.coef32[0];
    a.c1 = g.coef32[1];
    a.c2 = g.coef32[2];
    a.s2 = g.s2;
    a.vscale = std::ldexp(1.0, 2 * g.s2_exp);
    a.prior = g.c;
    a.ei_c = ei_c ? *ei_c : 0.0;
    float* e = ei_c ? (float*)ei : nullptr;
    rc = by_d_rec<1>((g.d + 2 + 3) / 4, [&](auto Sc) {
      constexpr int S = decltype(Sc)::value;
      if constexpr (S > (SCOOT_MAX_DIM + 5) / 4) {
        return fail(SCOOT_ERR_UNSUPPORTED, "posterior: d exceeds SCOOT_MAX_DIM");
      } else {
        return run32_by_rows<S>(g, Xc, n, (float*)mu, (float*)sigma, e, a, s);
      }
    });
  } else {
    Post64 a{};
    a.n = n;
    a.d = g.d;
    a.warp = g.warp && !xc_warped ? 1 : 0;
    for (int k = 0; k < SCOOT_MAX_DIM; ++k) {
      a.wa[k] = g.warp_a[k];
      a.wb[k] = g.warp_b[k];
    }
    a.nb16 = g.m_pad / kBlk16;
    a.plan = plan_rows16(a.nb16, posterior_waves(g.nb));
    for (int e = 0; e < 8; ++e)
      if (a.plan.nrows[e] > kMaxRows16) return fail(SCOOT_ERR_UNSUPPORTED, "posterior: row plan does not pack");
    for (int k = 0; k < SCOOT_MAX_DIM; ++k) a.scale[k] = g.scale64[k];
    a.c0 = g.coef64[0];
    a.c1 = g.coef64[1];
    a.c2 = g.coef64[2];
    a.s2 = g.s2;
    a.prior = g.c;
    a.ei_c = ei_c ? *ei_c : 0.0;
    double* e = ei_c ? (double*)ei : nullptr;
    rc = by_d_rec<1>(g.d, [&](auto Dc) {
      constexpr int D = decltype(Dc)::value;
      double *m64 = (double*)mu, *s64 = (double*)sigma;
      if (posterior_waves(g.nb) == 8) return run64<8, D>(g, Xc, n, m64, s64, e, a, s);
      return run64<4, D>(g, Xc, n, m64, s64, e, a, s);
    });
  }
  if (rc != SCOOT_OK) return rc;
  hipError_t err = hipGetLastError();
  if (err != hipSuccess) return fail(SCOOT_ERR_DEVICE, std::string("posterior launch: ") + hipGetErrorString(err));
  return SCOOT_OK;
}

}  // namespace scoot

// Sequential Kriging-believer selection of q candidates, an extension of the
// parallel suggestion of Sec. 4.6 (the paper takes the top k by EHVI at once).
//
// Each pick x_p joins the observations with the fantasy value y = mu(x_p) and
// the observation noise tau^2; the mean does not move (the fantasy equals it),
// the variance drops, the front gains the fantasy, and the next pick maximises
// EHVI over the feasible, not yet picked candidates.
//
// The variance after k picks, from the posterior of the observations alone:
//   C_p(x)   = k(x, x_p) - beta_p . k(x, X),  beta_p = K^-1 k(X, x_p)
//   w(x)     = L_S^-1 C(x),   L_S L_S^T = [C_p(x_p')] + tau^2 I
//   sigma^2  = sigma_0^2 - |w|^2
// so a candidate needs its m covariances once and k dot products with them,
// and nothing is kept per candidate between the picks.
//
// Only candidates that can win are scored again.  EHVI never grows from one
// pick to the next: the hypervolume improvement is convex in every objective
// (along one axis its slope is minus the open cross-section, which shrinks as
// the axis grows), so a smaller variance at the same mean lowers its
// expectation, and a larger front lowers it everywhere.  Hence every score
// computed earlier is an upper bound.  Per pick the seven best by bound are
// scored, the best of them is a lower bound on the maximum, and exactly the
// candidates whose bound reaches it (less a slack for rounding) are scored
// too; the pick is the maximum over all bounds, ties to the lowest index.  On
// the workloads (2^20 candidates, front of about 30) that is tens to a few
// thousand candidates per pick instead of the pool: a suggestion of eight
// took 12.4 ms when every pick streamed V = L^-1 K*^T (4.3 GB) from memory.
//
// A small pool is scored whole at every pick: w of every pick is kept, so a pick
// costs the covariances once more and a shorter chain of launches (kb_direct).
//
// Where many candidates score alike the list is long.  A bound that equals the
// best score cannot beat it, nor win the tie from a higher index, so such a
// candidate is not listed (all scores zero, or a pool far from every
// observation).  A list longer than kListed is not scored: a sample of it is,
// whose best is a better guess, and a second list holds what can still win
// against that.  Everything that decides is a set, so that the order in which
// the lists fill does not show.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstdint>
#include <cstring>
#include <type_traits>
#include <utility>
#include <vector>

#include "internal.h"
#include "select.h"

namespace scoot {

namespace {

typedef float f4_t __attribute__((ext_vector_type(4)));
typedef double d4_t __attribute__((ext_vector_type(4)));
typedef unsigned u4_t __attribute__((ext_vector_type(4)));

constexpr int kTop = 8;     // candidates of a selection: the pick and the next round's first guesses
constexpr int kPicks = 8;   // picks whose covariances one pass over the observations makes
constexpr int kListed = 16384;   // the longest list scored without waiting for its length
// More candidates than this are taken 64 to a wave: a workgroup of that form for
// every compute unit.
constexpr int64_t kWide = 65536;
// The same for a pass of one pick, all objectives counted: 160 of 256 compute units.
constexpr int64_t kWideOne = 40960;
constexpr double kSlack = 1e-4;  // of the best score, against rounding of the bounds

// One objective: its GP, the pool as the GP sees it, and what the picks left.
struct KbGp {
  const unsigned char* linv;  // units of L^-1 (pack_linv_f32)
  const double* xq;           // augmented observation rows
  const float* xc;            // pool, n x d, after input warping
  const float* mu;            // n
  const float* sd0;           // n: sigma of the observations alone
  double* v;                  // m_pad: L^-1 k(X, x) of the newest pick
  double* beta;               // q x m_pad
  double* ls;                 // q x q: rows of L_S
  float* w;                   // kb_w_rows x ld: w of earlier picks
  float* mu_list;             // outputs, per list entry
  float* sd_list;
  float* sd_out;              // n
  double scale[SCOOT_MAX_DIM];
  double c0d, c1d, c2d, s2, tau2;
  double vscale, bscale;  // 2^-s2_exp for products with linv, 4^s2_exp for beta beside covariances
  float c0, c1, c2;       // divided by 4^s2_exp
  int m, nj, nb32, m_pad, S;
};
struct KbArgs {
  KbGp g[SCOOT_MAX_OBJECTIVES];
  const int64_t* picks;  // device, in order
  int64_t ld;            // row stride of w: the pool's length, or of the first guesses
  int d, q, p;
};

// k(x, y) in double from scaled coordinates' squared distance.
__device__ inline double kb_cov(const KbGp& g, double r2) {
  const double u = sqrt(r2);
  return fma(u, fma(u, g.c2d, g.c1d), g.c0d) * exp2(-u);
}
// Scaled component k of observation i, from the augmented rows (they hold
// twice the coordinate, in the order pack_obs_f32 documents).
__device__ inline double kb_obs(const KbGp& g, int i, int k) {
  const int r = i & 15, t = 4 * (r & 3) + (r >> 2);
  return 0.5 * g.xq[((size_t)(i >> 4) * g.S + (k >> 2)) * 64 + 16 * (k & 3) + t];
}
// Eight consecutive entries of a row of 2^s2_exp L^-1 (the lane's, of one unit).
__device__ inline void kb_unit(const KbGp& g, int unit, int lane, double (&a)[8]) {
  const u4_t* at = reinterpret_cast<const u4_t*>(g.linv + (size_t)unit * 3 * 64 * 16) + lane;
  const u4_t p0 = at[0], p1 = at[64], p2 = at[128];
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    auto lo = [](unsigned w) { return (double)__builtin_bit_cast(float, w << 16); };
    auto hi = [](unsigned w) { return (double)__builtin_bit_cast(float, w & 0xffff0000u); };
    a[2 * i] = (lo(p2[i]) + lo(p1[i])) + lo(p0[i]);
    a[2 * i + 1] = (hi(p2[i]) + hi(p1[i])) + hi(p0[i]);
  }
}
__device__ inline int kb_unit_index(const KbGp& g, int j, int P) {
  return j * g.nb32 - (j - 1) * (j - 1) / 4 + g.nb32 - 1 - P;
}

// What the host reads back after a selection: the pick (-1: none), how many
// candidates were listed for it, its score and its means (the fantasies).
struct KbInfo {
  int64_t pick;
  int32_t count;
  float score, mu[SCOOT_MAX_OBJECTIVES];
};

// The pick, of a selection (idx given) or of the best key that scoring the
// guesses and a list has found, unless that list was too long to be scored: it
// joins the list of picks and leaves the pool, the host's figures are gathered,
// and the list is emptied.
__global__ void kb_pick_kernel(const KbArgs a, const int64_t* __restrict__ idx, const float* __restrict__ score,
                               const unsigned long long* __restrict__ top, int64_t cap, int k,
                               uint8_t* __restrict__ elig, int64_t* __restrict__ picks, KbInfo* __restrict__ info,
                               int32_t* __restrict__ count) {
  const int t = threadIdx.x;
  const int32_t listed = count[0];
  const Key64 key{*top};
  int64_t pick = idx ? idx[0] : (key.zero() ? -1 : key_index(key));
  if (listed > cap) pick = -1;
  __syncthreads();  // the count is read
  if (t == 0) {
    info->pick = pick;
    info->count = listed;
    info->score = idx ? score[0] : key_score(key);
    count[0] = 0;
    if (pick >= 0) {
      picks[k] = pick;
      elig[pick] = 0;
    }
  }
  if (t < a.p && pick >= 0) info->mu[t] = a.g[t].mu[pick];
}
__global__ void kb_zero_kernel(int32_t* count) { count[0] = 0; }

// v = L^-1 k(X, x_k), one row block of 32 per workgroup.
__global__ __launch_bounds__(256) void kb_v_kernel(const KbArgs a, int k) {
  const KbGp& g = a.g[blockIdx.y];
  __shared__ double ks[SCOOT_MAX_OBS + 32];
  __shared__ double part[4][32];
  const int P = blockIdx.x;
  if (P >= g.nb32) return;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const float* x = g.xc + a.picks[k] * a.d;
  const int cols = min(32 * P + 32, g.nj * 16);
  for (int i = tid; i < cols; i += 256) {
    double r2 = 0.0;
    for (int q = 0; q < a.d; ++q) {
      const double t = (double)x[q] * g.scale[q] - kb_obs(g, i, q);
      r2 = fma(t, t, r2);
    }
    ks[i] = i < g.m ? kb_cov(g, r2) : 0.0;
  }
  __syncthreads();
  double acc = 0.0;
  for (int j = wave; j < min(2 * P + 2, g.nj); j += 4) {
    double l[8];
    kb_unit(g, kb_unit_index(g, j, P), lane, l);
#pragma unroll
    for (int i = 0; i < 8; ++i) acc = fma(l[i], ks[16 * j + 8 * (lane >> 5) + i], acc);
  }
  acc += __shfl_xor(acc, 32);
  if (lane < 32) part[wave][lane] = acc;
  __syncthreads();
  if (tid < 32)
    g.v[32 * P + tid] = g.vscale * ((part[0][tid] + part[1][tid]) + (part[2][tid] + part[3][tid]));
}

// beta_k = L^-T v, a block of 16 columns.
__device__ inline void kb_beta(const KbGp& g, int j, int k) {
  __shared__ double part[4][16];
  if (j >= g.nj) return;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  double acc[8] = {};
  for (int P = j / 2 + wave; P < g.nb32; P += 4) {
    double l[8];
    kb_unit(g, kb_unit_index(g, j, P), lane, l);
    const double v = g.v[32 * P + (lane & 31)];
#pragma unroll
    for (int i = 0; i < 8; ++i) acc[i] = fma(l[i], v, acc[i]);
  }
#pragma unroll
  for (int i = 0; i < 8; ++i) {
    for (int o = 16; o >= 1; o >>= 1) acc[i] += __shfl_xor(acc[i], o);
    if ((lane & 31) == 0) part[wave][8 * (lane >> 5) + i] = acc[i];
  }
  __syncthreads();
  if (tid < 16)
    g.beta[(size_t)k * g.m_pad + 16 * j + tid] =
        g.vscale * ((part[0][tid] + part[1][tid]) + (part[2][tid] + part[3][tid]));
}

// Row k of L_S.  C_p(x_k) = k(x_k, x_p) - beta_p . k(X, x_k), where
// k(X, x_k) . beta_p = (L v_k) . (L^-T v_p): the covariances are made again.
__device__ inline void kb_chol(const KbArgs& a, const KbGp& g, int k) {
  __shared__ double ks[SCOOT_MAX_OBS + 32];
  __shared__ double row[SCOOT_MAX_Q + 1];
  __shared__ double var[4];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const float* x = g.xc + a.picks[k] * a.d;
  double s = 0.0;
  for (int i = tid; i < g.m; i += 256) {
    double r2 = 0.0;
    for (int q = 0; q < a.d; ++q) {
      const double t = (double)x[q] * g.scale[q] - kb_obs(g, i, q);
      r2 = fma(t, t, r2);
    }
    ks[i] = kb_cov(g, r2);
    s = fma(g.v[i], g.v[i], s);
  }
  for (int o = 32; o >= 1; o >>= 1) s += __shfl_xor(s, o);
  if (lane == 0) var[wave] = s;
  __syncthreads();
  // sixteen lanes to a pick: the dot product, and a dimension of the distance each
  static_assert(SCOOT_MAX_DIM <= 16, "a lane per dimension");
  const int c = tid & 15;
  for (int p = tid >> 4; p < k; p += 16) {
    const double* beta = g.beta + (size_t)p * g.m_pad;
    double dot = 0.0;
#pragma unroll 4
    for (int i = c; i < g.m; i += 16) dot = fma(beta[i], ks[i], dot);
    const double t = c < a.d ? ((double)x[c] - (double)g.xc[a.picks[p] * a.d + c]) * g.scale[c] : 0.0;
    double r2 = t * t;
    for (int o = 8; o >= 1; o >>= 1) {
      dot += __shfl_xor(dot, o);
      r2 += __shfl_xor(r2, o);
    }
    if (c == 0) row[p] = kb_cov(g, r2) - dot;
  }
  __syncthreads();
  if (wave != 0) return;
  // Forward substitution against the rows before, one wave: lane t holds what is
  // left of entry t, and entry p, once known, is taken off the later ones.  The
  // columns come eight at a time, ahead of their use.
  const double* lr = g.ls + (size_t)min(lane, max(k - 1, 0)) * a.q;
  double rest = lane < k ? row[lane] : 0.0;
  const double inv = lane < k ? 1.0 / lr[lane] : 0.0;
  double mine = 0.0, sum2 = 0.0;
  for (int p0 = 0; p0 < k; p0 += 8) {
    double col[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) col[u] = lane < k && lane > p0 + u ? lr[p0 + u] : 0.0;
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      if (p0 + u < k) {
        const double y = rest * inv;
        const double l = __hiloint2double(__builtin_amdgcn_readlane(__double2hiint(y), p0 + u),
                                          __builtin_amdgcn_readlane(__double2loint(y), p0 + u));
        if (lane == p0 + u) mine = l;
        rest = fma(-l, col[u], rest);
        sum2 = fma(l, l, sum2);
      }
    }
  }
  if (lane < k) g.ls[(size_t)k * a.q + lane] = mine;
  if (lane == 0) {
    const double prior = g.s2 - ((var[0] + var[1]) + (var[2] + var[3]));
    g.ls[(size_t)k * a.q + k] = sqrt(fmax(prior, 0.0) + g.tau2 - fmin(sum2, fmax(prior, 0.0)));
  }
}

// Both need v and not each other: the last workgroup of a row takes the latter.
__global__ __launch_bounds__(256) void kb_join_kernel(const KbArgs a, int k) {
  const KbGp& g = a.g[blockIdx.y];
  if (blockIdx.x + 1 < gridDim.x) kb_beta(g, (int)blockIdx.x, k);
  else kb_chol(a, g, k);
}

// sigma after the picks below k1, of a list (list or list64 given; the results
// go beside it) or of the pool: n entries or (live given) *live, none if that is
// more than n.  KP picks to a pass over the observations: kPicks from pick 0 on,
// or one, k1 - 1, with the w of the picks before it in rows, where its own joins
// them.  NARROW: 16 candidates per workgroup, its four waves sharing the
// observations (and the rows), w in LDS; otherwise 64 candidates per wave, w
// stored where a pass follows.  K* as in the posterior (distances on the fp64
// matrix cores), the dot products in double.  Bound (whole pool, m = 512, eight
// picks): the covariances, as in the posterior.
template <int S, bool NARROW, int KP>
__global__ __launch_bounds__(256, 2) void kb_sigma_kernel(const KbArgs a, const int32_t* __restrict__ list,
                                                          const int64_t* __restrict__ list64,
                                                          const int32_t* __restrict__ live, int64_t n, int k1) {
  constexpr int NT = NARROW ? 1 : 4;
  constexpr int NP = KP == 1 && NARROW ? 2 : KP;  // sums: KP covariances, and with rows sum w^2
  const KbGp& g = a.g[blockIdx.y];
  if (g.S != S) return;
  extern __shared__ __align__(16) unsigned char smem[];
  double* beta_l = reinterpret_cast<double*>(smem);  // [nj][KP][16]; NARROW: [4 waves][16][NP]
  double* w_l = beta_l + 4 * 16 * NP;                // NARROW: [picks][16]
  const int tid = threadIdx.x, lane = tid & 63, gr = lane >> 4, c = lane & 15;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int64_t base = NARROW ? (int64_t)blockIdx.x * 16 : (int64_t)blockIdx.x * 256 + wave * 64;
  if constexpr (NARROW) {
    if (live) n = *live <= n ? *live : 0;
    if (base >= n) return;
  }
  int64_t cand[NT];
  double bq[NT][S];
#pragma unroll
  for (int t = 0; t < NT; ++t) {
    const int64_t e = min(base + t * 16 + c, n - 1);
    cand[t] = e;
    if (list64) cand[t] = max(list64[e], (int64_t)0);
    else if (list) cand[t] = list[e];
    double nrm = 0.0;
#pragma unroll
    for (int s = 0; s < S; ++s) {
      const int k = 4 * s + gr;
      bq[t][s] = k < a.d ? (double)g.xc[cand[t] * a.d + k] * g.scale[min(k, SCOOT_MAX_DIM - 1)] : 0.0;
      nrm = fma(bq[t][s], bq[t][s], nrm);
    }
    nrm += __shfl_xor(nrm, 16);
    nrm += __shfl_xor(nrm, 32);
#pragma unroll
    for (int s = 0; s < S; ++s) {
      const int k = 4 * s + gr;
      if (k >= a.d) bq[t][s] = k == a.d ? 1.0 : (k == a.d + 1 ? nrm : 0.0);
    }
  }
  // the candidate that this lane finishes; wide: lane group gr finishes tile gr
  const int64_t e = NARROW ? base + c : base + lane;
  int64_t x;
  if constexpr (NARROW) {
    x = cand[0];
  } else {
    x = min(e, n - 1);
    if (list) x = list[x];
  }
  const bool mine = e < n && (!NARROW || (wave == 0 && gr == 0));
  double var = 0.0;
  if (mine) {
    const double s0 = (double)g.sd0[x];
    var = s0 * s0;
  }
  for (int b = KP == 1 ? k1 - 1 : 0; b < k1; b += KP) {
    const int kn = min(KP, k1 - b);
    if (KP > 1 && b > 0) __syncthreads();  // the pass before: its sums or beta are read, its w is written
    if constexpr (!NARROW) {
      for (int i = tid; i < g.nj * 16 * KP; i += 256) {
        const int j = i / (16 * KP), p = (i / 16) % KP;
        beta_l[i] = p < kn ? g.bscale * g.beta[(size_t)(b + p) * g.m_pad + 16 * j + (i & 15)] : 0.0;
      }
      __syncthreads();
    }
    double acc[NT][NP];
#pragma unroll
    for (int t = 0; t < NT; ++t)
#pragma unroll
      for (int p = 0; p < NP; ++p) acc[t][p] = 0.0;
    if constexpr (NARROW) {
      // k(x, x_p), one pick per lane group (the waves' sums are added below)
      const int p = wave * 4 + gr;
      if (p < kn) {
        const float* xr = g.xc + cand[0] * a.d;
        const float* xp = g.xc + a.picks[b + p] * a.d;
        double r2 = 0.0;
        for (int q = 0; q < a.d; ++q) {
          const double t = ((double)xr[q] - (double)xp[q]) * g.scale[q];
          r2 = fma(t, t, r2);
        }
        const double kx = kb_cov(g, r2);
#pragma unroll
        for (int q = 0; q < KP; ++q) acc[0][q] = q == p ? kx : 0.0;
      }
      // the earlier picks' w, one per lane group
      const int64_t at = min(base + c, n - 1);
      for (int t = p; t < b; t += 16) {
        const double w = KP == 1 ? (double)g.w[(size_t)t * a.ld + at] : w_l[t * 16 + c];
#pragma unroll
        for (int q = 0; q < KP; ++q)
          if (q < kn) acc[0][q] = fma(-g.ls[(size_t)(b + q) * a.q + t], w, acc[0][q]);
        if constexpr (KP == 1) acc[0][1] = fma(-w, w, acc[0][1]);
      }
    }
    for (int j = NARROW ? wave : 0; j < g.nj; j += NARROW ? 4 : 1) {
      double aq[S];
#pragma unroll
      for (int s = 0; s < S; ++s) aq[s] = (g.xq + (size_t)j * S * 64)[(unsigned)(s * 64 + lane)];
      double kv[NT][4];
#pragma unroll
      for (int t = 0; t < NT; ++t) {
        d4_t cr = d4_t{0.0, 0.0, 0.0, 0.0};
#pragma unroll
        for (int s = 0; s < S; ++s) cr = __builtin_amdgcn_mfma_f64_16x16x4f64(aq[s], bq[t][s], cr, 0, 0, 0);
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const float u = __builtin_amdgcn_sqrtf(fmaxf((float)(-cr[r]), 0.0f));
          kv[t][r] = (double)(fmaf(u, fmaf(u, g.c2, g.c1), g.c0) * __builtin_amdgcn_exp2f(-u));
        }
      }
#pragma unroll
      for (int p = 0; p < KP; ++p) {
        if (p < kn) {
          d4_t bv;
          if constexpr (NARROW)
            bv = g.bscale * *reinterpret_cast<const d4_t*>(g.beta + (size_t)(b + p) * g.m_pad + 16 * j + 4 * gr);
          else
            bv = *reinterpret_cast<const d4_t*>(beta_l + (j * KP + p) * 16 + 4 * gr);
#pragma unroll
          for (int t = 0; t < NT; ++t)
#pragma unroll
            for (int r = 0; r < 4; ++r) acc[t][p] = fma(-bv[r], kv[t][r], acc[t][p]);
        }
      }
    }
    // the lane groups' shares; NARROW: the waves' too
#pragma unroll
    for (int t = 0; t < NT; ++t)
#pragma unroll
      for (int p = 0; p < NP; ++p) {
        acc[t][p] += __shfl_xor(acc[t][p], 16);
        acc[t][p] += __shfl_xor(acc[t][p], 32);
      }
    double C[NP];
    if constexpr (NARROW) {
      if (gr == 0)
#pragma unroll
        for (int p = 0; p < NP; ++p) beta_l[(wave * 16 + c) * NP + p] = acc[0][p];
      __syncthreads();
#pragma unroll
      for (int p = 0; p < NP; ++p)
        C[p] = (beta_l[c * NP + p] + beta_l[(16 + c) * NP + p]) + (beta_l[(32 + c) * NP + p] + beta_l[(48 + c) * NP + p]);
    } else {
#pragma unroll
      for (int p = 0; p < NP; ++p)
        C[p] = gr == 0 ? acc[0][p]
                       : (gr == 1 ? acc[NT > 1 ? 1 : 0][p] : (gr == 2 ? acc[NT > 2 ? 2 : 0][p] : acc[NT - 1][p]));
    }
    if (!mine) continue;
    if constexpr (KP == 1 && NARROW) var += C[1];
#pragma unroll
    for (int p = 0; p < KP; ++p) {
      if (p < kn) {
        const double* l = g.ls + (size_t)(b + p) * a.q;
        double w = C[p];
        if constexpr (!NARROW) {
          const float* xr = g.xc + x * a.d;
          const float* xp = g.xc + a.picks[b + p] * a.d;
          double r2 = 0.0;
          for (int q = 0; q < a.d; ++q) {
            const double t = ((double)xr[q] - (double)xp[q]) * g.scale[q];
            r2 = fma(t, t, r2);
          }
          w += kb_cov(g, r2);
          for (int t0 = 0; t0 < b; t0 += 8) {  // eight loads in flight
            float wt[8];
#pragma unroll
            for (int t = 0; t < 8; ++t) wt[t] = g.w[(size_t)min(t0 + t, b - 1) * a.ld + e];
#pragma unroll
            for (int t = 0; t < 8; ++t) {
              const double wd = t0 + t < b ? (double)wt[t] : 0.0;
              w = fma(-l[min(t0 + t, b - 1)], wd, w);
              if constexpr (KP == 1) var = fma(-wd, wd, var);
            }
          }
        }
#pragma unroll
        for (int t = 0; t < p; ++t) w = fma(-l[b + t], C[t], w);
        C[p] = w / l[b + p];
        var = fma(-C[p], C[p], var);
        if constexpr (NARROW && KP > 1) w_l[(b + p) * 16 + c] = C[p];
        if (KP == 1 || (!NARROW && b + KP < k1)) g.w[(size_t)(b + p) * a.ld + e] = (float)C[p];
      }
    }
  }
  if (!mine) return;
  const float sd = (float)sqrt(fmax(var, 0.0));
  if (list || list64) {
    g.sd_list[e] = sd;
    g.mu_list[e] = g.mu[x];
  } else {
    g.sd_out[e] = sd;
  }
}

// The largest key of a wave, on every lane.
__device__ inline unsigned long long kb_wave_max(unsigned long long key) {
  for (int o = 32; o >= 1; o >>= 1) {
    const unsigned long long other = __shfl_xor(key, o);
    key = other > key ? other : key;
  }
  return key;
}

// Lists the candidates that can still win: eligible, and a bound that beats the
// best of the first guesses (kTop - 1, at idx) or comes within the slack of it,
// but for exact ties.  !FIRST: a bound that beats top, the best key that scoring
// the guesses and the sample has found, and a hash of the index of at most limit.
// Entries past cap are counted only.  One addition to the count per workgroup
// and 1024 candidates: with one per wave, where every wave lists something, the
// additions to one address were the kernel's time (n = 2^20: 65-120 us, now 8).
constexpr int kCompact = 4;  // candidates per thread
template <bool FIRST>
__global__ __launch_bounds__(256) void kb_compact_kernel(const float* __restrict__ bound,
                                                         const uint8_t* __restrict__ elig, int64_t n,
                                                         const int64_t* __restrict__ idx,
                                                         const float* __restrict__ first, uint32_t limit,
                                                         unsigned long long* __restrict__ top,
                                                         int32_t* __restrict__ list, int64_t cap,
                                                         int32_t* __restrict__ count) {
  __shared__ int in_wave[4];
  __shared__ int start;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  unsigned long long key = 0;
  float best = -INFINITY;
  if (FIRST) {
    if (lane < kTop - 1 && idx[lane] >= 0 && first[lane] == first[lane]) {
      best = first[lane];
      key = make_key(best, idx[lane], true).v;
    }
    key = kb_wave_max(key);
    for (int o = 32; o >= 1; o >>= 1) best = fmaxf(best, __shfl_xor(best, o));
    if (blockIdx.x == 0 && threadIdx.x == 0) *top = 0;  // scoring raises it
  } else {
    key = *top;
  }
  const float thr = fabsf(best) < INFINITY ? best - (float)kSlack * fabsf(best) : best;
  for (int64_t c0 = (int64_t)blockIdx.x * 256 * kCompact; c0 < n; c0 += (int64_t)gridDim.x * 256 * kCompact) {
    const int64_t i = c0 + (int64_t)threadIdx.x * kCompact;
    float b[kCompact] = {};
    uint8_t e[kCompact] = {};
    if (i + kCompact <= n) {  // both arrays are 256-byte aligned
      *reinterpret_cast<f4_t*>(b) = *reinterpret_cast<const f4_t*>(bound + i);
      *reinterpret_cast<uint32_t*>(e) = *reinterpret_cast<const uint32_t*>(elig + i);
    } else {
      for (int t = 0; t < kCompact && i + t < n; ++t) {
        b[t] = bound[i + t];
        e[t] = elig[i + t];
      }
    }
    unsigned in = 0;
#pragma unroll
    for (int t = 0; t < kCompact; ++t) {
      const uint32_t x = (uint32_t)i + t;
      if (e[t] != 0 && b[t] == b[t] && (make_key(b[t], i + t, true).v > key || (FIRST && b[t] >= thr && b[t] != best)) &&
          (FIRST || x * 2654435761u <= limit))
        in |= 1u << t;
    }
    int at = __popc(in);  // entries up to this lane's last
    for (int o = 1; o < 64; o <<= 1) {
      const int v = __shfl_up(at, o);
      if (lane >= o) at += v;
    }
    if (lane == 63) in_wave[wave] = at;
    __syncthreads();
    const int sum = in_wave[0] + in_wave[1] + in_wave[2] + in_wave[3];
    if (threadIdx.x == 0 && sum) start = atomicAdd(count, sum);
    __syncthreads();
    int64_t to = (int64_t)at - __popc(in);
    if (sum) {
      to += start;
      for (int w = 0; w < wave; ++w) to += in_wave[w];
    }
#pragma unroll
    for (int t = 0; t < kCompact; ++t)
      if ((in >> t & 1u) && to < cap) list[to++] = (int32_t)(i + t);
    __syncthreads();  // in_wave and start are read
  }
}

// The scores of the list (as many entries as kb_sigma takes), and of the first
// guesses (idx given), become their candidates' bounds, and the best of them top.
__global__ __launch_bounds__(256) void kb_scatter_kernel(const int32_t* __restrict__ list,
                                                         const int32_t* __restrict__ live, int n,
                                                         const float* __restrict__ val,
                                                         const int64_t* __restrict__ idx,
                                                         const float* __restrict__ first, float* __restrict__ bound,
                                                         unsigned long long* __restrict__ top) {
  const int i = blockIdx.x * 256 + threadIdx.x;
  if (live) n = *live <= n ? *live : 0;
  unsigned long long key = 0;
  auto set = [&](int64_t x, float score) {
    bound[x] = score;
    const unsigned long long mine = make_key(score, x, true).v;
    key = mine > key ? mine : key;
  };
  if (idx && i < kTop - 1 && idx[i] >= 0) set(idx[i], first[i]);  // a guess on the list: the same score twice
  if (i < n) set(list[i], val[i]);
  key = kb_wave_max(key);
  if ((threadIdx.x & 63) == 0 && key) atomicMax(top, key);
}

constexpr size_t kKbAlign = 256;
size_t align256(size_t b) { return (b + kKbAlign - 1) / kKbAlign * kKbAlign; }

struct KbLayout {
  size_t mu, sd, bound, elig, votes, list, mu_list, sd_list, val, w, xw;  // of the pool's size
  size_t idx, score, first, nvalid, picks, info, count, top, v, beta, ls;  // small
  size_t total;
};

// Whether every pick scores the whole pool, in a chain of six launches.  The
// other way's twelve cost some 30 us a pick more whatever the pool, and the
// first guesses and the list go over all the picks before; a pool's pass costs
// the covariances and about 64 of them more per candidate and objective for the
// scores and w.  Both sides, ms: p = 1, m = 256, n = 131,072, q = 4 0.34 and
// 0.41, q = 32 2.4 and 4.0; p = 3, m = 64, n = 262,144, q = 9 1.23 and 1.12, q =
// 64 9.3 and 10.1; p = 2, m = 512, n = 262,144, q = 32 8.3 and 6.2.
bool kb_direct(const GPDevice* const* g, int p, int64_t n, int q) {
  int64_t each = 0;
  for (int j = 0; j < p; ++j) each += (g[j]->m + 15) / 16 * 16 + 64;
  return n <= ((int64_t)(72 + 5 * q / 2) << 20) / each;
}
// Rows of w that are kept: of every pick that a score carries, or of those but
// for the last chunk.
int kb_w_rows(const GPDevice* const* g, int p, int64_t n, int q) {
  if (kb_direct(g, p, n, q)) return q - 1;
  return q > 2 ? (q - 2) / kPicks * kPicks : 0;
}

KbLayout kb_layout(const GPDevice* const* g, int p, int64_t n, int q) {
  KbLayout L{};
  size_t off = 0;
  auto take = [&](size_t bytes) {
    const size_t at = off;
    off += align256(bytes);
    return at;
  };
  size_t m_pad = 0, xw = 0;
  for (int j = 0; j < p; ++j) {
    m_pad = std::max(m_pad, (size_t)g[j]->m_pad);
    xw += g[j]->warp ? align256((size_t)n * g[j]->d * 4) : 0;  // the pool after each warped GP's input warping
  }
  L.mu = take((size_t)p * n * 4);
  L.sd = take((size_t)p * n * 4);
  L.bound = take((size_t)n * 4);
  L.elig = take((size_t)n);
  L.votes = take((size_t)n * 4);
  L.list = take((size_t)n * 4);
  L.mu_list = take((size_t)p * std::max<int64_t>(n, kTop) * 4);
  L.sd_list = take((size_t)p * std::max<int64_t>(n, kTop) * 4);
  L.val = take((size_t)std::max<int64_t>(n, kTop) * 4);
  L.w = take((size_t)p * kb_w_rows(g, p, n, q) * std::max<int64_t>(n, kTop) * 4);
  L.xw = take(xw);
  L.idx = take(kTop * 8);
  L.score = take(kTop * 4);
  L.first = take(kTop * 4);
  L.nvalid = take(4);
  L.picks = take((size_t)q * 8);
  L.info = take(sizeof(KbInfo));
  L.count = take(4);
  L.top = take(8);
  L.v = take((size_t)p * m_pad * 8);
  L.beta = take((size_t)p * q * m_pad * 8);
  L.ls = take((size_t)p * q * q * 8);
  L.total = off;
  return L;
}

template <int S, bool NARROW, int KP>
int launch_sigma_s(const KbArgs& a, const int32_t* list, const int64_t* list64, const int32_t* live, int64_t n, int k1,
                   hipStream_t s) {
  auto kern = kb_sigma_kernel<S, NARROW, KP>;
  int nj = 0;
  for (int j = 0; j < a.p; ++j) nj = std::max(nj, a.g[j].nj);
  // [4 waves][16][sums] and w, or beta
  const size_t lds = NARROW ? (size_t)(4 * 16 * (KP == 1 ? 2 : KP) + (KP == 1 ? 0 : k1 * 16)) * 8 : (size_t)nj * 16 * KP * 8;
  const int rc = allow_full_lds((const void*)kern, "believer");
  if (rc != SCOOT_OK) return rc;
  const int64_t blocks = NARROW ? (n + 15) / 16 : (n + 255) / 256;
  hipLaunchKernelGGL(kern, dim3((unsigned)blocks, (unsigned)a.p), dim3(256), lds, s, a, list, list64, live, n, k1);
  return SCOOT_OK;
}

// one: pick k1 - 1 over the whole pool, from the rows of w before it.
int launch_sigma(const KbArgs& a, const int32_t* list, const int64_t* list64, const int32_t* live, int64_t n, int k1,
                 bool one, hipStream_t s) {
  if (n == 0) return SCOOT_OK;
  const bool narrow = live || list64 || (one ? a.p * n <= kWideOne : n <= kWide);
  auto launch = [&](auto S) {
    constexpr int s_ = decltype(S)::value;
    if (one)
      return narrow ? launch_sigma_s<s_, true, 1>(a, list, list64, live, n, k1, s)
                    : launch_sigma_s<s_, false, 1>(a, list, list64, live, n, k1, s);
    return narrow ? launch_sigma_s<s_, true, kPicks>(a, list, list64, live, n, k1, s)
                  : launch_sigma_s<s_, false, kPicks>(a, list, list64, live, n, k1, s);
  };
  switch (a.g[0].S) {  // the GPs share d
    case 1: return launch(std::integral_constant<int, 1>());
    case 2: return launch(std::integral_constant<int, 2>());
    case 3: return launch(std::integral_constant<int, 3>());
    case 4: return launch(std::integral_constant<int, 4>());
    default: return launch(std::integral_constant<int, 5>());
  }
}

}  // namespace

// With room to place the parts on 256-byte boundaries wherever the workspace
// starts: they are read by 16 bytes and hold counters.
size_t kb_workspace_bytes(const GPDevice* const* g, int p, int64_t n, int q) {
  return kb_layout(g, p, n, q).total + kKbAlign - 1;
}

int run_kriging_believer(const GPDevice* const* g, int p, const ForestDevice* f, const uint8_t* known,
                         int64_t vote_min, const float* Xc, int64_t n, const double* Y_obs, int m_obs,
                         const double* ref, int q, void* ws, int64_t* picks, double* pick_acq, int* n_picked,
                         float* mu_out, float* sigma_out, void* stream) {
  hipStream_t s = (hipStream_t)stream;
  const KbLayout L = kb_layout(g, p, n, q);
  unsigned char* w = (unsigned char*)(((uintptr_t)ws + kKbAlign - 1) / kKbAlign * kKbAlign);
  float* mu = (float*)(w + L.mu);
  float* sd = (float*)(w + L.sd);
  float* bound = (float*)(w + L.bound);
  uint8_t* elig = (uint8_t*)(w + L.elig);
  int32_t* votes = (int32_t*)(w + L.votes);
  int32_t* list = (int32_t*)(w + L.list);
  float* val = (float*)(w + L.val);
  int64_t* idx = (int64_t*)(w + L.idx);
  float* score = (float*)(w + L.score);
  float* first = (float*)(w + L.first);
  int32_t* nvalid = (int32_t*)(w + L.nvalid);
  int64_t* picks_d = (int64_t*)(w + L.picks);
  KbInfo* info_d = (KbInfo*)(w + L.info);
  int32_t* count_d = (int32_t*)(w + L.count);
  unsigned long long* top = (unsigned long long*)(w + L.top);
  const int64_t nl = std::max<int64_t>(n, kTop);
  const bool direct = kb_direct(g, p, n, q);
  int m_pad = 0;
  for (int j = 0; j < p; ++j) m_pad = std::max(m_pad, g[j]->m_pad);

  KbArgs a{};
  a.picks = picks_d;
  a.ld = nl;
  a.d = g[0]->d;
  a.q = q;
  a.p = p;
  const void *mus[SCOOT_MAX_OBJECTIVES], *sds[SCOOT_MAX_OBJECTIVES], *mul[SCOOT_MAX_OBJECTIVES],
      *sdl[SCOOT_MAX_OBJECTIVES];
  size_t xoff = L.xw;
  int rc;
  for (int j = 0; j < p; ++j) {
    KbGp& o = a.g[j];
    o.linv = (const unsigned char*)g[j]->linv;
    o.xq = (const double*)g[j]->xs;
    o.xc = Xc;
    if (g[j]->warp) {  // the pool as this GP sees it
      float* xw = (float*)(w + xoff);
      xoff += align256((size_t)n * g[j]->d * 4);
      rc = launch_warp_pool(*g[j], Xc, n, xw, stream);
      if (rc != SCOOT_OK) return rc;
      o.xc = xw;
    }
    o.mu = mu + (size_t)j * n;
    o.sd0 = sd + (size_t)j * n;
    o.v = (double*)(w + L.v) + (size_t)j * m_pad;
    o.beta = (double*)(w + L.beta) + (size_t)j * q * m_pad;
    o.ls = (double*)(w + L.ls) + (size_t)j * q * q;
    o.w = (float*)(w + L.w) + (size_t)j * kb_w_rows(g, p, n, q) * nl;
    o.mu_list = (float*)(w + L.mu_list) + (size_t)j * nl;
    o.sd_list = (float*)(w + L.sd_list) + (size_t)j * nl;
    // where every pick scores the pool: sigma after the picks, beside no list
    o.sd_out = direct ? o.sd_list : sigma_out ? sigma_out + (size_t)j * n : nullptr;
    for (int k = 0; k < SCOOT_MAX_DIM; ++k) o.scale[k] = g[j]->scale64[k];
    o.c0d = g[j]->coef64[0];
    o.c1d = g[j]->coef64[1];
    o.c2d = g[j]->coef64[2];
    o.vscale = std::ldexp(1.0, -g[j]->s2_exp);
    o.bscale = std::ldexp(1.0, 2 * g[j]->s2_exp);
    o.c0 = g[j]->coef32[0];
    o.c1 = g[j]->coef32[1];
    o.c2 = g[j]->coef32[2];
    o.s2 = g[j]->s2;
    o.tau2 = g[j]->tau2;
    o.m = g[j]->m;
    o.nj = (g[j]->m + 15) / 16;
    o.nb32 = g[j]->nb;
    o.m_pad = m_pad;
    o.S = (g[j]->d + 2 + 3) / 4;
    mus[j] = o.mu;
    sds[j] = o.sd0;
    mul[j] = o.mu_list;
    sdl[j] = o.sd_list;
    rc = launch_posterior(*g[j], o.xc, n, mu + (size_t)j * n, sd + (size_t)j * n, nullptr, nullptr, stream, true);
    if (rc != SCOOT_OK) return rc;
  }
  rc = f ? launch_forest(*f, Xc, n, vote_min, votes, elig, nullptr, stream, known)
         : launch_mask_init(elig, known, n, stream);
  if (rc != SCOOT_OK) return rc;

  auto device_error = [](hipError_t e) {
    return fail(SCOOT_ERR_DEVICE, std::string("believer: ") + hipGetErrorString(e));
  };
  // the front so far: the observations first, then the front and the fantasies
  std::vector<double> front(Y_obs, Y_obs + (size_t)m_obs * p);
  int nb32 = 0, nj = 0;
  for (int j = 0; j < p; ++j) {
    nb32 = std::max(nb32, a.g[j].nb32);
    nj = std::max(nj, a.g[j].nj);
  }
  *n_picked = 0;
  for (int k = 0; k < q; ++k) {
    BoxTable bt;
    rc = build_boxes(front.data(), (int)(front.size() / p), p, ref, bt);
    if (rc != SCOOT_OK) return rc;
    KbInfo info{};
    // One read-back per pick: what the next round needs of it is made while the
    // host builds that round's boxes.
    auto pick = [&](const int64_t* selected, int64_t cap) {
      hipLaunchKernelGGL(kb_pick_kernel, dim3(1), dim3(64), 0, s, a, selected, score, top, cap, k, elig, picks_d, info_d,
                         count_d);
      hipError_t e = hipGetLastError();
      if (e == hipSuccess) e = hipMemcpyAsync(&info, info_d, sizeof info, hipMemcpyDeviceToHost, s);
      if (e == hipSuccess) e = hipStreamSynchronize(s);
      return e == hipSuccess ? SCOOT_OK : device_error(e);
    };
    if (k == 0) {
      hipLaunchKernelGGL(kb_zero_kernel, dim3(1), dim3(1), 0, s, count_d);
      rc = launch_ehvi_topq(mus, sds, p, n, SCOOT_F32, bt, bound, elig, direct ? 1 : kTop, idx, score, nvalid, stream);
      if (rc == SCOOT_OK) rc = pick(idx, n);
    } else if (direct) {
      rc = launch_ehvi_topq(mus, sdl, p, n, SCOOT_F32, bt, bound, elig, 1, idx, score, nvalid, stream);
      if (rc == SCOOT_OK) rc = pick(idx, n);
    } else {
      const dim3 blocks((unsigned)std::min<int64_t>((n + 256 * kCompact - 1) / (256 * kCompact), 2048));
      auto score_list = [&](const int32_t* live, int64_t entries, const int64_t* guesses) {
        int rc = launch_sigma(a, list, nullptr, live, entries, k, false, s);
        if (rc == SCOOT_OK) rc = launch_ehvi(mul, sdl, p, entries, SCOOT_F32, bt, val, stream);
        if (rc == SCOOT_OK && entries > 0)
          hipLaunchKernelGGL(kb_scatter_kernel, dim3((unsigned)((entries + 255) / 256)), dim3(256), 0, s, list, live,
                             (int)entries, val, guesses, first, bound, top);
        return rc;
      };
      // A second list, of what beats top: limit of 2^32 - 1 of it.
      auto second_list = [&](uint32_t limit, int64_t most) {
        hipLaunchKernelGGL(kb_compact_kernel<false>, blocks, dim3(256), 0, s, bound, elig, n, nullptr, nullptr, limit,
                           top, list, most, count_d);
      };
      // The first guesses: the best bounds after the last pick.  The length of
      // the list that they leave stays on the device until the pick.
      const int64_t cap = std::min<int64_t>(n, kListed);
      rc = launch_sigma(a, nullptr, idx + 1, nullptr, kTop - 1, k, false, s);
      if (rc == SCOOT_OK) rc = launch_ehvi(mul, sdl, p, kTop - 1, SCOOT_F32, bt, first, stream);
      if (rc != SCOOT_OK) return rc;
      hipLaunchKernelGGL(kb_compact_kernel<true>, blocks, dim3(256), 0, s, bound, elig, n, idx + 1, first, 0u, top,
                         list, cap, count_d);
      rc = score_list(count_d, cap, idx + 1);
      if (rc == SCOOT_OK) rc = pick(nullptr, cap);
      if (rc == SCOOT_OK && info.count > cap) {
        second_list((uint32_t)((uint64_t)cap * 0x80000000u / (uint64_t)info.count), cap);  // about cap / 2
        rc = score_list(count_d, cap, nullptr);
        if (rc != SCOOT_OK) return rc;
        hipLaunchKernelGGL(kb_zero_kernel, dim3(1), dim3(1), 0, s, count_d);
        second_list(UINT32_MAX, n);
        int32_t count = 0;
        hipError_t e = hipGetLastError();
        if (e == hipSuccess) e = hipMemcpyAsync(&count, count_d, sizeof count, hipMemcpyDeviceToHost, s);
        if (e == hipSuccess) e = hipStreamSynchronize(s);
        if (e != hipSuccess) return device_error(e);
        rc = score_list(nullptr, count, nullptr);
        if (rc == SCOOT_OK) rc = pick(nullptr, n);
      }
    }
    if (rc != SCOOT_OK) return rc;
    if (info.pick < 0) break;
    picks[k] = info.pick;
    if (pick_acq) pick_acq[k] = info.score;
    *n_picked = k + 1;
    if (k + 1 == q) break;
    front = std::move(bt.front);
    for (int j = 0; j < p; ++j) front.push_back((double)info.mu[j]);
    hipLaunchKernelGGL(kb_v_kernel, dim3((unsigned)nb32, (unsigned)p), dim3(256), 0, s, a, k);
    hipLaunchKernelGGL(kb_join_kernel, dim3((unsigned)nj + 1, (unsigned)p), dim3(256), 0, s, a, k);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return device_error(e);
    rc = SCOOT_OK;
    if (direct)
      rc = launch_sigma(a, nullptr, nullptr, nullptr, n, k + 1, true, s);
    else if (k > 0)
      rc = launch_topq(bound, elig, n, SCOOT_F32, kTop - 1, idx + 1, score + 1, nvalid, stream);
    if (rc != SCOOT_OK) return rc;
  }
  // the posterior the last scoring round saw (mu never moves; sigma carries
  // the picks before that round)
  hipError_t e = hipSuccess;
  if (mu_out) e = hipMemcpyAsync(mu_out, mu, (size_t)p * n * 4, hipMemcpyDeviceToDevice, s);
  if (e == hipSuccess && sigma_out) {
    const int seen = *n_picked == q ? q - 1 : *n_picked;
    if (seen == 0 || direct) {
      for (int j = 0; j < p && e == hipSuccess; ++j)
        e = hipMemcpyAsync(sigma_out + (size_t)j * n, seen ? a.g[j].sd_list : a.g[j].sd0, (size_t)n * 4,
                           hipMemcpyDeviceToDevice, s);
    } else {
      rc = launch_sigma(a, nullptr, nullptr, nullptr, n, seen, false, s);
      if (rc != SCOOT_OK) return rc;
      e = hipGetLastError();
    }
  }
  if (e != hipSuccess) return device_error(e);
  return SCOOT_OK;
}

}  // namespace scoot

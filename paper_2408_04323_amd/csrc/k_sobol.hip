// Candidate generation on the device: a Sobol pool on the search space's
// grids, and the known-constraint mask (Sec. 4.5.3: the optimiser's space is
// pruned by constraints known beforehand; Sec. 4.7: missing suggestions are
// filled with Sobol points; Sec. 4.1 and Algorithm 1: the first observations
// are Sobol points; the engines' rules are listed in the appendix on known
// constraints).
//
// Sobol points (Sobol 1967, direction numbers by the recurrence of Bratley and
// Fox 1988, Gray-code order of Antonov and Saleev 1979): coordinate j of point
// i is the XOR of V_j[k] over the set bits k of gray(i) = i ^ (i >> 1), over
// 2^32.  Consecutive points differ by one direction number: point i + 1 is
// point i XOR V_j[ctz(i + 1)].  A thread owns one dimension of a run of 16
// points whose first index is a multiple of 16, so inside the run the
// direction numbers it needs are V_j[0..3] in a fixed order; only the run's
// first point is built bit by bit.  The block's points are staged row-major
// in LDS and leave in coalesced stores; the known-constraint rows are
// evaluated on the staged float32 values in the same pass.
//
// Grids: level count L >= 2 rounds u to rint(u (L - 1)) / (L - 1) in double
// (half to even), L = 1 is a boolean (1 when u >= 1/2), L = 0 is continuous;
// the result is stored as float32.  A candidate is admissible when every
// constraint row sum_k A[r][k] x_k <= b[r] holds, the sum taken over k in
// order in double with each product and each sum rounded separately.  Linear
// rows express every rule the paper lists: an order between two knobs, two
// switches that exclude each other, one switch that requires another, and a
// bound that applies unless a boolean is set (big-M on the boolean).
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstring>
#include <string>
#include <type_traits>

#include "internal.h"

namespace scoot {

namespace {

constexpr int kSobolThreads = 256;
constexpr int kSobolRun = 16;       // points per thread; runs start at multiples of 16
constexpr int kSobolBits = 32;
// Workgroups of a large pool: six per compute unit (eight take the same time), each
// loading the direction numbers once and looping over chunks of 256 / d runs.
constexpr int kSobolBlocks = 256 * 6;

struct Constraints {
  double A[SCOOT_MAX_CONSTRAINTS * SCOOT_MAX_DIM];  // row-major r x d
  double b[SCOOT_MAX_CONSTRAINTS];
  int r, d;
};

struct SobolArgs {
  uint32_t v[kSobolBits * SCOOT_MAX_DIM];  // [k][j]: direction number k of dimension j (k-major, stride d)
  int32_t levels[SCOOT_MAX_DIM];
  double step[SCOOT_MAX_DIM];   // 1 / (levels - 1) of the grids that a product rounds exactly, 0 for the others
  Constraints con;
  int64_t n;
  int64_t row0;   // pool row of the first run's first point: -(skip mod 16)
  uint64_t first; // Sobol index of that point: skip - (skip mod 16)
  int nbits;      // bit length of the last index generated
  int64_t chunks; // of 256 / d runs
};
static_assert(sizeof(SobolArgs) <= 4096, "kernel arguments are limited to 4 KiB");

// One coordinate on its grid, rint(u q) / q in double and then float, q =
// levels - 1.  The division is a product with 1 / q wherever that gives the
// same float: with k / q in [2^e, 2^(e + 1)) the product is off by at most
// 2^(e - 51), and k / q is at least 2^(e - 24) / q away from the nearest midpoint
// of two floats, or is that midpoint, odd 2^(e - 24) with odd >= 2^24, which
// takes k >= 2^24; so q < 2^24 has neither.  A continuous coordinate (s = 2^-32,
// no rounding) and a boolean (the top bit, q = 1) take the same steps, so that
// the lanes of a wave, which hold different dimensions, do not diverge.
struct Snap {
  unsigned shift;  // 31 for a boolean
  double scale;    // of the integer: 2^-32 q, 1 for a boolean
  bool grid;
  double step;     // 1 / q, 0: divide by q
  double q;
};
__device__ inline Snap snap_of(int L, double step) {
  if (L == 0) return Snap{0, 0x1p-32, false, 1.0, 1.0};
  if (L == 1) return Snap{31, 1.0, false, 1.0, 1.0};
  const double q = (double)(L - 1);
  return Snap{0, q * 0x1p-32, true, step, q};
}
template <bool DIVIDE>
__device__ inline float snapped(uint32_t x, const Snap& s) {
  double v = (double)(x >> s.shift) * s.scale;
  v = s.grid ? rint(v) : v;
  if (DIVIDE && s.step == 0.0) return (float)(v / s.q);
  return (float)(v * s.step);
}

// Sequential, separately rounded row sums (no fused multiply-add); the
// candidate's d coordinates are read once.
template <int D>
__device__ inline bool admissible(const float* x, const Constraints& c) {
#pragma clang fp contract(off)
  float xv[D];
#pragma unroll
  for (int k = 0; k < D; ++k) xv[k] = x[k];
  bool ok = true;
  for (int r = 0; r < c.r; ++r) {
    double s = 0.0;
#pragma unroll
    for (int k = 0; k < D; ++k) s = s + c.A[r * D + k] * (double)xv[k];
    ok = ok && s <= c.b[r];
  }
  return ok;
}

// Bound: the writes, 4 d + 1 bytes a candidate (2^20 candidates, d = 12, two
// constraint rows: 51 MB, 10 us at a copy's rate).  Measured there: 19 us; 35 us
// with a division per grid coordinate, branches between the three kinds of
// knob, dimension counts known at run time only and one float per store.
template <int D, bool DIVIDE>
__global__ __launch_bounds__(kSobolThreads) void sobol_pool_kernel(float* __restrict__ Xc, uint8_t* __restrict__ known,
                                                                   const SobolArgs a) {
  constexpr int R = kSobolThreads / D;        // runs of a chunk
  constexpr int kPts = R * kSobolRun;
  constexpr int kRow = (kSobolRun + 1) * D;   // a run in LDS: one spare point, so that runs start on different banks
  __shared__ uint32_t vs[kSobolBits * D];
  __shared__ __align__(16) float tile[R * kRow];  // point (run, t) at run kRow + t D
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  for (int i = tid; i < kSobolBits * D; i += kSobolThreads) vs[i] = a.v[i];
  __syncthreads();
  const int run = tid / D, j = tid - run * D;
  const uint32_t v0 = vs[j], v1 = vs[D + j], v2 = vs[2 * D + j], v3 = vs[3 * D + j];
  const Snap snap = snap_of(a.levels[j], a.step[j]);

  for (int64_t chunk = blockIdx.x; chunk < a.chunks; chunk += gridDim.x) {
    if (run < R) {
      const uint64_t i0 = a.first + ((uint64_t)chunk * R + run) * kSobolRun;
      const uint64_t g = i0 ^ (i0 >> 1);
      uint32_t x = 0;
      for (int k = 3; k < a.nbits; ++k) x ^= vs[k * D + j] & (0u - (uint32_t)((g >> k) & 1u));  // i0 ends in four zeros
      float* out = tile + run * kRow + j;
#pragma unroll
      for (int t = 0; t < kSobolRun; ++t) {
        out[t * D] = snapped<DIVIDE>(x, snap);
        if (t + 1 < kSobolRun) {
          const int c = __builtin_ctz(t + 1);  // 0..3, fixed at compile time
          x ^= c == 0 ? v0 : c == 1 ? v1 : c == 2 ? v2 : v3;
        }
      }
    }
    __syncthreads();

    const int64_t row_base = a.row0 + chunk * kPts;
    float* to = Xc + row_base * D;
    // By 16 bytes where the chunk is whole and aligned, else by element.  From
    // seven dimensions on a run per wave at a time, without a division; a run of
    // fewer would leave most lanes idle (n = 2^24, one run per wave and flat: d =
    // 9 unaligned 182 and 217 us, d = 1 aligned 49 and 32).
    if (row_base >= 0 && row_base + kPts <= a.n && ((uintptr_t)to & 15) == 0) {
      if constexpr (D >= 7) {
        // 4 D <= 64 vectors of four floats per run
        for (int rr = wave; rr < R; rr += kSobolThreads / 64) {
          if (lane < 4 * D) {
            const float* from = tile + rr * kRow + 4 * lane;
            reinterpret_cast<float4*>(to)[rr * 4 * D + lane] = float4{from[0], from[1], from[2], from[3]};
          }
        }
      } else {
        for (int v = tid; v < R * 4 * D; v += kSobolThreads) {
          const float* from = tile + 4 * v + v / (4 * D) * D;
          reinterpret_cast<float4*>(to)[v] = float4{from[0], from[1], from[2], from[3]};
        }
      }
    } else {
      const int64_t lo = -row_base * D, hi = (a.n - row_base) * D;
      if constexpr (D >= 7) {
        for (int rr = wave; rr < R; rr += kSobolThreads / 64)
#pragma unroll
          for (int i = 0; i < (kSobolRun * D + 63) / 64; ++i) {
            const int e = i * 64 + lane, at = rr * kSobolRun * D + e;
            if (e < kSobolRun * D && at >= lo && at < hi) to[at] = tile[rr * kRow + e];
          }
      } else {
        for (int e = tid; e < kPts * D; e += kSobolThreads)
          if (e >= lo && e < hi) to[e] = tile[e + e / (kSobolRun * D) * D];
      }
    }
    if (known) {
      for (int p = tid; p < kPts; p += kSobolThreads) {
        const int64_t row = row_base + p;
        if (row >= 0 && row < a.n)
          known[row] = admissible<D>(tile + p / kSobolRun * kRow + p % kSobolRun * D, a.con) ? 1 : 0;
      }
    }
    __syncthreads();  // the tile is read
  }
}

// The same for a dimension count known at run time only.
__device__ inline bool admissible_row(const float* x, const Constraints& c) {
#pragma clang fp contract(off)
  bool ok = true;
  for (int r = 0; r < c.r; ++r) {
    double s = 0.0;
    for (int k = 0; k < c.d; ++k) s = s + c.A[r * c.d + k] * (double)x[k];
    ok = ok && s <= c.b[r];
  }
  return ok;
}

__global__ __launch_bounds__(256) void known_constraints_kernel(const float* __restrict__ Xc, int64_t n,
                                                                uint8_t* __restrict__ known, const Constraints c) {
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
    known[i] = admissible_row(Xc + i * c.d, c) ? 1 : 0;
}

__global__ void mask_init_kernel(uint8_t* __restrict__ mask, const uint8_t* __restrict__ known, int64_t n) {
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
    mask[i] = known ? (known[i] != 0 ? 1 : 0) : 1;
}

int check_constraints(const double* A, const double* b, int r, int d, Constraints& c) {
  if (r < 0 || r > SCOOT_MAX_CONSTRAINTS)
    return fail(SCOOT_ERR_UNSUPPORTED, "known constraints: r must be in 0..SCOOT_MAX_CONSTRAINTS");
  if (r > 0 && (!A || !b)) return fail(SCOOT_ERR_INVALID_ARG, "known constraints: null A or b");
  std::memset(&c, 0, sizeof(c));
  c.r = r;
  c.d = d;
  for (int i = 0; i < r * d; ++i) {
    if (!std::isfinite(A[i])) return fail(SCOOT_ERR_INVALID_ARG, "known constraints: non-finite A");
    c.A[i] = A[i];
  }
  for (int i = 0; i < r; ++i) {
    if (std::isnan(b[i])) return fail(SCOOT_ERR_INVALID_ARG, "known constraints: NaN b");
    c.b[i] = b[i];
  }
  return SCOOT_OK;
}

// Direction numbers V[k] = m_k 2^(32 - k), k = 1..32, of the dimension with
// primitive polynomial `poly` (bit t = coefficient of x^t; degree s = its bit
// length - 1) and initial values m_1..m_s.  Beyond s, m_k is the XOR of
// 2^t a_t m_(k-t) over t = 1..s-1 (a_t the coefficient of x^(s-t)) with
// m_(k-s) and 2^s m_(k-s).
int direction_numbers(uint32_t poly, const uint32_t* vinit, uint32_t* V) {
  if (poly == 0 || (poly & 1u) == 0) return fail(SCOOT_ERR_INVALID_ARG, "sobol: polynomial must have constant term 1");
  int s = 31;
  while (!((poly >> s) & 1u)) --s;
  if (s > SCOOT_SOBOL_MAX_DEGREE) return fail(SCOOT_ERR_UNSUPPORTED, "sobol: polynomial degree above SCOOT_SOBOL_MAX_DEGREE");
  uint64_t m[kSobolBits + 1];
  for (int k = 1; k <= kSobolBits; ++k) {
    if (s == 0) {
      m[k] = 1;
    } else if (k <= s) {
      m[k] = vinit[k - 1];
      if ((m[k] & 1u) == 0 || m[k] >= ((uint64_t)1 << k))
        return fail(SCOOT_ERR_INVALID_ARG, "sobol: initial value m_k must be odd and below 2^k");
    } else {
      uint64_t v = m[k - s] ^ (m[k - s] << s);
      for (int t = 1; t < s; ++t)
        if ((poly >> (s - t)) & 1u) v ^= m[k - t] << t;
      m[k] = v;
    }
  }
  for (int k = 1; k <= kSobolBits; ++k) V[k - 1] = (uint32_t)(m[k] << (kSobolBits - k));
  return SCOOT_OK;
}

// f(std::integral_constant<int, d>{}) for the d in 1..SCOOT_MAX_DIM given at run time.
template <int D, typename F>
void dispatch_dim(int d, F&& f) {
  if constexpr (D <= SCOOT_MAX_DIM) {
    if (d == D) return f(std::integral_constant<int, D>{});
    dispatch_dim<D + 1>(d, f);
  }
}

int launched(const char* what) {
  hipError_t err = hipGetLastError();
  if (err != hipSuccess) return fail(SCOOT_ERR_DEVICE, std::string(what) + ": " + hipGetErrorString(err));
  return SCOOT_OK;
}

}  // namespace

int launch_sobol_pool(const uint32_t* poly, const uint32_t* vinit, int d, const int32_t* levels, int64_t skip,
                      int64_t n, const double* A, const double* b, int r, float* Xc, uint8_t* known, void* stream) {
  if (d < 1 || d > SCOOT_MAX_DIM) return fail(SCOOT_ERR_INVALID_ARG, "sobol: d must be in 1..SCOOT_MAX_DIM");
  if (!poly || !vinit || !levels) return fail(SCOOT_ERR_INVALID_ARG, "sobol: null poly, vinit or levels");
  if (n < 0 || skip < 0 || skip + n > ((int64_t)1 << 32))
    return fail(SCOOT_ERR_INVALID_ARG, "sobol: need n >= 0, skip >= 0, skip + n <= 2^32");
  if (n > 0 && !Xc) return fail(SCOOT_ERR_INVALID_ARG, "sobol: null Xc");
  SobolArgs a;
  std::memset(&a, 0, sizeof(a));
  int rc = check_constraints(A, b, r, d, a.con);
  if (rc != SCOOT_OK) return rc;
  bool divide = false;
  for (int j = 0; j < d; ++j) {
    if (levels[j] < 0) return fail(SCOOT_ERR_INVALID_ARG, "sobol: negative level count");
    a.levels[j] = levels[j];
    a.step[j] = levels[j] >= 2 && levels[j] <= (1 << 24) ? 1.0 / (double)(levels[j] - 1) : 0.0;
    divide = divide || levels[j] > (1 << 24);
    uint32_t V[kSobolBits];
    rc = direction_numbers(poly[j], vinit + (size_t)j * SCOOT_SOBOL_MAX_DEGREE, V);
    if (rc != SCOOT_OK) return rc;
    for (int k = 0; k < kSobolBits; ++k) a.v[k * d + j] = V[k];
  }
  if (n == 0) return SCOOT_OK;
  const uint64_t last = (uint64_t)(skip + n - 1);
  a.nbits = 1;
  while (a.nbits < kSobolBits && (last >> a.nbits) != 0) ++a.nbits;
  a.n = n;
  a.row0 = -(skip & (kSobolRun - 1));
  a.first = (uint64_t)skip - (uint64_t)(skip & (kSobolRun - 1));
  const int64_t runs = (n - a.row0 + kSobolRun - 1) / kSobolRun;
  a.chunks = (runs + kSobolThreads / d - 1) / (kSobolThreads / d);
  const dim3 grid((unsigned)std::min<int64_t>(a.chunks, kSobolBlocks));
  dispatch_dim<1>(d, [&](auto D) {
    if (divide)
      hipLaunchKernelGGL((sobol_pool_kernel<decltype(D)::value, true>), grid, dim3(kSobolThreads), 0,
                         (hipStream_t)stream, Xc, known, a);
    else
      hipLaunchKernelGGL((sobol_pool_kernel<decltype(D)::value, false>), grid, dim3(kSobolThreads), 0,
                         (hipStream_t)stream, Xc, known, a);
  });
  return launched("sobol launch");
}

int launch_known_constraints(const float* Xc, int64_t n, int d, const double* A, const double* b, int r,
                             uint8_t* known, void* stream) {
  if (d < 1 || d > SCOOT_MAX_DIM) return fail(SCOOT_ERR_INVALID_ARG, "known constraints: d must be in 1..SCOOT_MAX_DIM");
  if (n < 0 || (n > 0 && (!Xc || !known))) return fail(SCOOT_ERR_INVALID_ARG, "known constraints: bad n or null pointer");
  Constraints c;
  int rc = check_constraints(A, b, r, d, c);
  if (rc != SCOOT_OK) return rc;
  if (n == 0) return SCOOT_OK;
  int64_t blocks = (n + 255) / 256;
  if (blocks > 8192) blocks = 8192;
  hipLaunchKernelGGL(known_constraints_kernel, dim3((unsigned)blocks), dim3(256), 0, (hipStream_t)stream, Xc, n, known,
                     c);
  return launched("known constraints launch");
}

int launch_mask_init(uint8_t* mask, const uint8_t* known, int64_t n, void* stream) {
  if (n == 0) return SCOOT_OK;
  int64_t blocks = (n + 255) / 256;
  if (blocks > 4096) blocks = 4096;
  hipLaunchKernelGGL(mask_init_kernel, dim3((unsigned)blocks), dim3(256), 0, (hipStream_t)stream, mask, known, n);
  return launched("mask launch");
}

}  // namespace scoot

// Subspace refresh of SubZero+: Haar-distributed factor of a Gaussian panel
// (Eq. 11, Alg. 1) -- thin QR with each column of Q multiplied by the sign of
// the matching diagonal entry of R, so the corrected R has diag(R) > 0.
//
// That corrected factor is the unique Q with Q^T Q = I and Omega = Q R,
// diag(R) > 0.  It is computed here by CholeskyQR2 in float64 (Fukaya,
// Nakatsukasa, Yanagisawa, Yamamoto, 2014): R1 = chol(Omega^T Omega),
// Q1 = Omega R1^-1, R2 = chol(Q1^T Q1), Q = Q1 R2^-1, R = R2 R1.  A Cholesky
// factor has a positive diagonal, so the sign correction is built in.  The
// second pass restores orthogonality to working precision.  What limits the
// method is a pivot of the first factorisation sinking into the rounding noise
// of the Gram matrix, which takes a column within ~1e-8 of the span of the
// earlier ones (column scaling alone does not: the relative pivots are scale
// free).  Gaussian panels, whose condition number is about
// (sqrt(rows) + sqrt(r)) / (sqrt(rows) - sqrt(r)), essentially never get there.
//
// Launches per call, each over every panel of the call (the panel descriptors sit in a table in
// the workspace, written by k_cqr_fill; a row launch's workgroup finds its panel by binary search
// over the table), all float64 with fixed-order sums (the result is bitwise reproducible):
//   rows 0   per chunk of rows: partial Omega^T Omega
//   chol     per panel: sum of the partials, Cholesky -> diag(R1), X1 = R1^-1
//   rows 1   per chunk: Q1 = Omega X1, partial Q1^T Q1
//   chol     per panel: R2, M = X1 R2^-1; diag(R) = diag(R2) diag(R1); info
//   rows 2   per chunk: Q = Omega M, written as fp32
// and, where the chunks are short (few panels), k_cqr_reduce before each chol: it adds a panel's
// partials on many CUs, which the one workgroup of chol would read at one CU's rate.
//
// The row passes run on v_mfma_f64_16x16x4_f64: the Gram matrix as sums of 4-row outer products
// over its upper 16 x 16 tiles, the products 16 rows at a time over the upper triangle of X1 or M
// (both triangular: column tile t takes the K blocks c <= t).
//
// Short and long chunks.  A chunk is one workgroup.  2048-row chunks leave most of the chip idle on
// a few panels (one OPT-13B layer: 50 workgroups; an OPT-1.3B layer at r = 128: 18), so a call with
// fewer than FEW_WG of them takes 512-row (r <= 64) or 256-row chunks.  Their partials go to the
// panel's own output Q, which nothing reads or writes before the last pass fills it (the
// workspace's size is a promise, and the no-allocation variant's scratch is fixed).  Where one output
// of the call overlaps an Omega, another output, diag(R) or info, or is smaller than its partials (few
// rows; any rows at r = 1 and at 65 <= r <= 72, whose tiles are padded to 128 columns), the whole call
// keeps the long chunks.  A panel's sum is the same tree either way (units of 128 or 256 rows, added in order within 2048 rows, then the
// 2048-row sums in order), so its Q is the same bits whatever else the call holds.
//
// Measured, whole call, before (a factorisation column by column in LDS, 2048- and 1024-row chunks,
// vector FMA for r > 64) and now: an OPT-13B layer's 12 panels at r = 64 631 -> 137 us (row passes
// 308 -> 78, factorisations 326 -> 48); an OPT-1.3B layer's at r = 128 2979 -> 253 us (row passes
// 1862 -> 126, factorisations 1106 -> 118); 480 OPT-13B panels 3149 -> 2031 us at r = 64 and
// 36.1 -> 6.5 ms at r = 128.
//
// A pivot that is not positive marks the panel rank deficient at that column
// (an exactly zero column gives a zero pivot): R's row there is zero, the Q
// column is zero, and the other columns are formed as if it were absent.
#include "zo_internal.h"

#include <algorithm>
#include <mutex>
#include <type_traits>
#include <vector>

namespace {

constexpr int CHUNK = 2048;       // rows per workgroup, long chunks
constexpr int UNIT = 128;         // r <= 64: rows per wave and unit of the summation tree
constexpr int FINE = 4 * UNIT;    // r <= 64: rows per workgroup, short chunks
constexpr int WUNIT = 256;        // r > 64: unit and short chunk
constexpr int FEW_WG = 512;
constexpr int FEW_PANELS = 64;
constexpr int FILL_PANELS = 48;   // descriptors per k_cqr_fill launch (kernel arguments)

typedef double f64x4 __attribute__((ext_vector_type(4)));

struct CqrPanel {
  const float* omega;
  float* q;
  float* r_diag;
  int* info;
  double* part;  // partial Gram matrices per chunk: the upper 16 x 16 tiles, row-major each
  double* R1;    // RP: diag(R1)
  double* X1;    // RP x RP: (R1^-1)^T
  double* M;     // RP x RP: (R1^-1 R2^-1)^T
  int rows, chunk_begin;
};
struct CqrArgs {
  const CqrPanel* p;  // the call's descriptor table (workspace)
  int count, r;
  int chunk;          // rows per chunk of this call (CHUNK, FINE or WUNIT)
};
struct CqrFill {
  CqrPanel p[FILL_PANELS];
  CqrPanel* dst;
  int n;
};

// Copies n host descriptors (kernel arguments) into the table, one 32-bit word per thread.
__global__ __launch_bounds__(256) void k_cqr_fill(CqrFill f) {
  constexpr int W = (int)(sizeof(CqrPanel) / 4);
  static_assert(sizeof(CqrPanel) % 4 == 0, "descriptor of whole words");
  const int x = blockIdx.x * 256 + threadIdx.x;
  if (x < f.n * W) ((uint32_t*)f.dst)[x] = ((const uint32_t*)f.p)[x];
}

// The panel that row workgroup wg belongs to: the last k with chunk_begin <= wg
// (chunk_begin is non-decreasing from 0; a panel without rows has no chunks).
__device__ __forceinline__ int find_panel(const CqrArgs& a, int wg) {
  int lo = 0, hi = a.count - 1;
  while (lo < hi) {
    const int mid = (lo + hi + 1) >> 1;
    if (a.p[mid].chunk_begin <= wg) lo = mid;
    else hi = mid - 1;
  }
  return lo;
}

__device__ __forceinline__ f64x4 mfma64(double a, double b, f64x4 c) {
  return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
}

// Upper tile p of RK x RK tiles in row-major order: its row and column.
constexpr int pair_row(int p, int RK) {
  int ta = 0;
  while (p >= RK - ta) { p -= RK - ta; ++ta; }
  return ta;
}
constexpr int pair_col(int p, int RK) {
  int ta = 0;
  while (p >= RK - ta) { p -= RK - ta; ++ta; }
  return ta + p;
}
constexpr int pair_idx(int ta, int tb, int RK) { return ta * RK - ta * (ta - 1) / 2 + (tb - ta); }

typedef float f32x4_a4 __attribute__((ext_vector_type(4), aligned(4)));

// Columns col .. col + 3 of a row of Omega, zero outside the panel's rows x r.
__device__ __forceinline__ f32x4 omega4(const CqrPanel& P, int row, int col, int r) {
  f32x4 v = {0.f, 0.f, 0.f, 0.f};
  if (row >= P.rows) return v;
  const float* o = P.omega + (size_t)row * r + col;
  if (col + 4 <= r) return (f32x4)*(const f32x4_a4*)o;
#pragma unroll
  for (int e = 0; e < 4; ++e)
    if (col + e < r) v[e] = o[e];
  return v;
}

// PASS 0: partial Omega^T Omega of this chunk.  PASS 1: partial Q1^T Q1 with
// Q1 = Omega X1.  PASS 2: Q = Omega M written as fp32.  Entries outside the
// panel's rows x r read as zero.  A Gram tile (ta <= tb) accumulates, per
// 4-row step, the MFMA of the rows' columns 16 ta + i (A) and 16 tb + j (B):
// lane l brings row base + l / 16, column 16 t + l % 16 as the operand of
// tile t.  A product 16 rows x RP takes the row's columns in blocks c of 16, element e of each
// lane's four in MFMA e: lane l multiplies column 16 c + 4 (l / 16) + e of row base + l % 16 with
// that row of X (any one-to-one map of (step, lane group) to columns sums the same terms).
// The product's output registers are, lane for lane, the operands of the Gram MFMAs of its
// rows (output lane l, register v holds row 4 v + l / 16, column l % 16), so Q1 never leaves the
// registers.  Bound by the fp64 MFMAs (2048 FLOP in 64 cycles).  A wave takes UNIT rows of a short
// chunk, four units of a long one; units, then waves, are added in order.
template <int RK, int PASS>
__global__ __launch_bounds__(256) void k_cqr_rows(CqrArgs a) {
  constexpr int RP = 16 * RK, NPAIR = RK * (RK + 1) / 2;
  constexpr int XP = RP + 2;  // pitch of X^T's rows: 16 rows at one 16-byte column on distinct banks
  __shared__ __attribute__((aligned(16))) double Mx[PASS == 0 ? 1 : RP * XP];
  __shared__ double red[PASS == 2 ? 1 : 4][PASS == 2 ? 1 : NPAIR * 256];  // each wave's sum of units
  const CqrPanel P = a.p[find_panel(a, blockIdx.x)];
  const int chunk = blockIdx.x - P.chunk_begin;
  const int r = a.r, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int l16 = lane & 15, g = lane >> 4;
  if (PASS >= 1) {
    const double* src = PASS == 1 ? P.X1 : P.M;
    for (int x = tid; x < RP * RP; x += 256) Mx[x / RP * XP + x % RP] = src[x];
    __syncthreads();
  }
  const int wrows = a.chunk / 4;
  // Omega entries as loaded (fp32, zero outside the panel); widened to float64 at use (exact).
  auto om = [&](int row, int col) -> float {
    return (row < P.rows && col < r) ? P.omega[(size_t)row * r + col] : 0.f;
  };
  f64x4 acc[NPAIR];
  // The Gram tiles over 4 rows whose tile-t operands are v[t].
  auto gram = [&](const double* v) {
    int p = 0;
#pragma unroll
    for (int ta = 0; ta < RK; ++ta)
#pragma unroll
      for (int tb = ta; tb < RK; ++tb, ++p) acc[p] = mfma64(v[ta], v[tb], acc[p]);
  };
  for (int u0 = 0; u0 < wrows; u0 += UNIT) {
    const int row0 = chunk * a.chunk + wave * wrows + u0;
    const int nrow = min(UNIT, P.rows - row0);  // this unit's rows (none past the end)
    if (nrow <= 0 && u0 > 0) break;
#pragma unroll
    for (int p = 0; p < NPAIR; ++p) acc[p] = (f64x4){0.0, 0.0, 0.0, 0.0};
    if (PASS == 0) {
      // 32 rows per step (eight 4-row Gram steps), the next step's loads issued before the MFMAs.
      float nx[8][RK];
      auto load = [&](int s) {
#pragma unroll
        for (int u = 0; u < 8; ++u)
#pragma unroll
          for (int t = 0; t < RK; ++t) nx[u][t] = om(row0 + s + 4 * u + g, 16 * t + l16);
      };
      if (nrow > 0) load(0);
      for (int s = 0; s < nrow; s += 32) {
        float cur[8][RK];
#pragma unroll
        for (int u = 0; u < 8; ++u)
#pragma unroll
          for (int t = 0; t < RK; ++t) cur[u][t] = nx[u][t];
        if (s + 32 < nrow) load(s + 32);
#pragma unroll
        for (int u = 0; u < 8; ++u) {
          double v[RK];
#pragma unroll
          for (int t = 0; t < RK; ++t) v[t] = (double)cur[u][t];
          gram(v);
        }
      }
    } else {
      f32x4 nx[RK];
      auto load = [&](int s) {
#pragma unroll
        for (int c = 0; c < RK; ++c) nx[c] = omega4(P, row0 + s + l16, 16 * c + 4 * g, r);
      };
      if (nrow > 0) load(0);
      for (int s = 0; s < nrow; s += 16) {
        f32x4 av[RK];
#pragma unroll
        for (int c = 0; c < RK; ++c) av[c] = nx[c];
        if (s + 16 < nrow) load(s + 16);
        // The RK product chains interleaved (each still sums its K steps in order).
        f64x4 q[RK];
#pragma unroll
        for (int t = 0; t < RK; ++t) q[t] = (f64x4){0.0, 0.0, 0.0, 0.0};
#pragma unroll
        for (int c = 0; c < RK; ++c) {
          double m[RK][4];
#pragma unroll
          for (int t = c; t < RK; ++t) {
            const double* x = &Mx[(16 * t + l16) * XP + 16 * c + 4 * g];
            const double2 m01 = *(const double2*)x, m23 = *(const double2*)(x + 2);
            m[t][0] = m01.x; m[t][1] = m01.y; m[t][2] = m23.x; m[t][3] = m23.y;
          }
#pragma unroll
          for (int e = 0; e < 4; ++e)
#pragma unroll
            for (int t = c; t < RK; ++t) q[t] = mfma64((double)av[c][e], m[t][e], q[t]);
        }
        // q[t][v]: row row0 + s + 4 v + g, column 16 t + l16.
        if (PASS == 1) {
#pragma unroll
          for (int v = 0; v < 4; ++v) {
            double w[RK];
#pragma unroll
            for (int t = 0; t < RK; ++t) w[t] = q[t][v];
            gram(w);
          }
        } else {
#pragma unroll
          for (int v = 0; v < 4; ++v) {
            const int row = row0 + s + 4 * v + g;
            if (row >= P.rows) continue;
#pragma unroll
            for (int t = 0; t < RK; ++t)
              if (16 * t + l16 < r) P.q[(size_t)row * r + 16 * t + l16] = (float)q[t][v];
          }
        }
      }
    }
    if (PASS != 2) {
#pragma unroll
      for (int p = 0; p < NPAIR; ++p)
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          double& d = red[wave][p * 256 + v * 64 + lane];
          d = u0 == 0 ? acc[p][v] : d + acc[p][v];
        }
    }
  }
  if (PASS == 2) return;
  __syncthreads();
  // The waves' sums added in wave order, written as the chunk's upper tiles.
  double* out = P.part + (size_t)chunk * NPAIR * 256;
  for (int x = tid; x < NPAIR * 256; x += 256) out[x] = ((red[0][x] + red[1][x]) + red[2][x]) + red[3][x];
}

// f(0), f(1), ... with constant arguments, so that register arrays keep constant indices.
template <int I, int N, typename F>
__device__ __forceinline__ void static_for(F& f) {
  if constexpr (I < N) {
    f(std::integral_constant<int, I>{});
    static_for<I + 1, N>(f);
  }
}

// The row passes for 64 < r <= 128 (RK = 8).  All 36 upper Gram tiles and the product of a
// 16-row group do not fit one wave's registers, so the 8 waves of a workgroup share 32 rows at a
// time: Omega's rows are staged in LDS (fp32); wave w forms column tile w of the first 16 rows and
// tile 7 - w of the last 16 (36 MFMAs each, whatever w), Q1 goes to LDS in float64; then wave w
// accumulates its 4 or 5 Gram tiles over all 32 rows (waves w and w + 4, which share a SIMD, have 9).
// X^T's 36 lower tiles sit in LDS with 18-double rows (conflict-free 16-byte reads).  At one
// workgroup per CU its 2 waves per SIMD keep the matrix cores fed through the three barriers of a
// step (9216 matrix cycles).  The vector-FMA kernel it replaces took 484 / 855 / 524 us for the
// three passes of an OPT-1.3B layer's panels (36864 rows x 128).
constexpr int WK = 8, WRP = 16 * WK, WPAIRS = WK * (WK + 1) / 2, WROWS = 32;
constexpr int WXT = 16 * 18;        // doubles per tile of X^T
constexpr int WOP = WRP + 4;        // pitch of the Omega rows (floats)
constexpr int WQP = WRP + 16;       // pitch of the Q1 rows (doubles)

template <int W>
struct WidePairs {  // Gram tiles of wave W
  static constexpr int P0 = W < 4 ? 9 * W : 9 * (W - 4) + 5;
  static constexpr int NP = W < 4 ? 5 : 4;
  static constexpr bool uses(int t) {
    for (int p = P0; p < P0 + NP; ++p)
      if (pair_row(p, WK) == t || pair_col(p, WK) == t) return true;
    return false;
  }
};

// acc += the wave's Gram tiles over the 32 staged rows; at(row, col) reads an entry.  A loop of one
// 4-row step: the eight waves run eight instances of it at once, which have to share the
// instruction cache.
template <int W, typename At>
__device__ __forceinline__ void wide_gram(f64x4* acc, At at, int g, int l16) {
  using S = WidePairs<W>;
#pragma unroll 2
  for (int s = 0; s < WROWS; s += 4) {
    double v[WK];
    auto read = [&](auto T) {
      constexpr int t = decltype(T)::value;
      if constexpr (S::uses(t)) v[t] = at(s + g, 16 * t + l16);
    };
    static_for<0, WK>(read);
    auto mul = [&](auto I) {
      constexpr int p = decltype(I)::value, ta = pair_row(S::P0 + p, WK), tb = pair_col(S::P0 + p, WK);
      acc[p] = mfma64(v[ta], v[tb], acc[p]);
    };
    static_for<0, S::NP>(mul);
  }
}

template <int PASS>
__global__ __launch_bounds__(512) void k_cqr_rows_wide(CqrArgs a) {
  __shared__ __attribute__((aligned(16))) float Om[WROWS * WOP];
  __shared__ __attribute__((aligned(16))) double Xt[PASS == 0 ? 2 : WPAIRS * WXT];
  __shared__ __attribute__((aligned(16))) double Q1[PASS == 1 ? WROWS * WQP : 2];
  const CqrPanel P = a.p[find_panel(a, blockIdx.x)];
  const int chunk = blockIdx.x - P.chunk_begin;
  const int r = a.r, tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int l16 = lane & 15, g = lane >> 4;
  if (PASS >= 1) {
    const double* src = PASS == 1 ? P.X1 : P.M;
    for (int x = tid; x < WRP * WRP; x += 512) {
      const int i = x / WRP, k = x % WRP, t = i >> 4, c = k >> 4;
      if (c <= t) Xt[(t * (t + 1) / 2 + c) * WXT + (i & 15) * 18 + (k & 15)] = src[x];
    }
  }
  const int base = chunk * a.chunk;
  const int rows = min(a.chunk, P.rows - base);
  f32x4 nx[2];
  auto load = [&](int s) {
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      const int x = tid + 512 * u;
      nx[u] = omega4(P, base + s + (x >> 5), 4 * (x & 31), r);
    }
  };
  f64x4 tot[5], acc[5];
#pragma unroll
  for (int p = 0; p < 5; ++p) tot[p] = acc[p] = (f64x4){0.0, 0.0, 0.0, 0.0};
  // Column tile t of staged rows h .. h + 15.
  auto product = [&](int h, int t) {
    f64x4 q = (f64x4){0.0, 0.0, 0.0, 0.0};
    for (int c = 0; c <= t; ++c) {
      const f32x4 o = *(const f32x4*)&Om[(h + l16) * WOP + 16 * c + 4 * g];
      const double* x = &Xt[(t * (t + 1) / 2 + c) * WXT + l16 * 18 + 4 * g];
      const double2 m01 = *(const double2*)x, m23 = *(const double2*)(x + 2);
      q = mfma64((double)o[0], m01.x, q);
      q = mfma64((double)o[1], m01.y, q);
      q = mfma64((double)o[2], m23.x, q);
      q = mfma64((double)o[3], m23.y, q);
    }
    return q;
  };
  if (rows > 0) load(0);
  for (int s = 0; s < rows; s += WROWS) {
    __syncthreads();  // the previous rows have been consumed (and, at first, X^T is staged)
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      const int x = tid + 512 * u;
      *(f32x4*)&Om[(x >> 5) * WOP + 4 * (x & 31)] = nx[u];
    }
    __syncthreads();
    if (s + WROWS < rows) load(s + WROWS);
    if (PASS >= 1) {
#pragma unroll
      for (int half = 0; half < 2; ++half) {
        const int h = 16 * half, t = half ? WK - 1 - wave : wave;
        const f64x4 q = product(h, t);
        const int col = 16 * t + l16;
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          const int row = h + 4 * v + g;
          if (PASS == 1)
            Q1[row * WQP + col] = q[v];
          else if (base + s + row < P.rows && col < r)
            P.q[(size_t)(base + s + row) * r + col] = (float)q[v];
        }
      }
      if (PASS == 2) continue;
      __syncthreads();
    }
    auto at = [&](int row, int col) -> double {
      if constexpr (PASS == 0) return (double)Om[row * WOP + col];
      else return Q1[row * WQP + col];
    };
    switch (wave) {
      case 0: wide_gram<0>(acc, at, g, l16); break;
      case 1: wide_gram<1>(acc, at, g, l16); break;
      case 2: wide_gram<2>(acc, at, g, l16); break;
      case 3: wide_gram<3>(acc, at, g, l16); break;
      case 4: wide_gram<4>(acc, at, g, l16); break;
      case 5: wide_gram<5>(acc, at, g, l16); break;
      case 6: wide_gram<6>(acc, at, g, l16); break;
      default: wide_gram<7>(acc, at, g, l16); break;
    }
    if ((s + WROWS) % WUNIT == 0 || s + WROWS >= rows) {  // the unit is complete
#pragma unroll
      for (int p = 0; p < 5; ++p) {
        tot[p] += acc[p];
        acc[p] = (f64x4){0.0, 0.0, 0.0, 0.0};
      }
    }
  }
  if (PASS == 2) return;
  const int p0 = wave < 4 ? 9 * wave : 9 * (wave - 4) + 5, np = wave < 4 ? 5 : 4;
  double* out = P.part + ((size_t)chunk * WPAIRS + p0) * 256 + lane;
#pragma unroll
  for (int p = 0; p < 5; ++p)
    if (p < np) {
#pragma unroll
      for (int v = 0; v < 4; ++v) out[p * 256 + v * 64] = tot[p][v];
    }
}

// Short chunks: the panel's partials added into its first one, a thread per entry: the chunks of
// each 2048 rows in order, then those sums in order (what the long chunks' passes add up to).
__global__ __launch_bounds__(256) void k_cqr_reduce(CqrArgs a, int npair) {
  const CqrPanel& P = a.p[blockIdx.y];
  const int nchunk = (P.rows + a.chunk - 1) / a.chunk, per = CHUNK / a.chunk;
  double* p = P.part + (size_t)blockIdx.x * 256 + threadIdx.x;
  const size_t step = (size_t)npair * 256;
  double sum = 0.0;
  for (int c = 0; c < nchunk; c += per) {
    double v[8];
#pragma unroll
    for (int k = 0; k < 8; ++k) v[k] = k < per && c + k < nchunk ? p[(c + k) * step] : 0.0;
    double s = v[0];
#pragma unroll
    for (int k = 1; k < 8; ++k) s += v[k];
    sum += s;
  }
  p[0] = sum;
}

// Sum of the panel's partials (chunk order), then Cholesky and the triangular inverse in one
// elimination.  With G = L D L^T (L unit lower, D the pivots d_k), R = D^1/2 L^T and
// R^-T = D^-1/2 L^-1, and L^-1 is what the row operations of the elimination make of the identity:
// step k takes f_i = G_ki / d_k times row k off every row i > k, of G and of the second matrix E.
// FINAL: this is R2 and E starts as X1^T, so it ends as D^-1/2 L^-1 X1^T = (X1 R2^-1)^T = M^T.
//
// A chain of r steps on one CU: what bounds it is the latency from one pivot row to the next.  So
// both matrices live in registers (one wave per column group: lane l has column l, and l + 64 for
// r > 64; rows dealt to H waves in turn) and a step is one barrier: the waves that own row k put it
// (and f = row / d) into LDS, everyone takes the row's entries of its own columns and the f_i of
// its own rows.  r = 64: 152 / 174 us for the two factorisations of a column-by-column kernel in
// LDS before; r = 128: 475 / 631 us.
//
// A pivot that is not positive gives f = 0 (no row is changed) and a zero row of D^-1/2, which
// zeroes exactly its column of R^-1 and, through f = 0, its row.
template <int RK, bool FINAL>
__global__ __launch_bounds__(RK > 4 ? 1024 : 512) void k_cqr_chol(CqrArgs a, int reduced) {
  constexpr int RP = 16 * RK, NPAIR = RK * (RK + 1) / 2;
  constexpr int NC = RP > 64 ? 2 : 1;  // columns per lane
  constexpr int H = NC == 2 ? 8 : 4;   // waves that share a column group's rows
  constexpr int NR = RP / H;           // rows per wave
  __shared__ __attribute__((aligned(16))) double fb[2][RP], gb[2][RP], eb[2][RP];
  __shared__ double piv[RP];
  __shared__ int bad;
  const CqrPanel& P = a.p[blockIdx.x];
  const int r = a.r, tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const bool isE = wave >= H;
  const int h = wave % H;
  if (tid == 0) bad = 0x7fffffff;
  for (int k = tid; k < RP; k += 128 * H) piv[k] = 0.0;
  double A[NR][NC];  // rows H ii + h, columns lane + 64 c
#pragma unroll
  for (int ii = 0; ii < NR; ++ii)
#pragma unroll
    for (int c = 0; c < NC; ++c) A[ii][c] = 0.0;
  if (!isE) {
    const int nchunk = reduced ? (P.rows > 0 ? 1 : 0) : (P.rows + a.chunk - 1) / a.chunk;
    // LB rows' loads of a chunk in flight together.
    constexpr int LB = NC == 2 ? 8 : NR;
    auto add = [&](auto I0) {
      constexpr int i0 = decltype(I0)::value;
      for (int ch = 0; ch < nchunk; ++ch) {
        const double* pc = P.part + (size_t)ch * NPAIR * 256;
        double v[LB][NC];
#pragma unroll
        for (int y = 0; y < LB; ++y)
#pragma unroll
          for (int c = 0; c < NC; ++c) {
            const int i = H * (i0 + y) + h, j = lane + 64 * c;
            v[y][c] = (i <= j && j < r) ? pc[pair_idx(i >> 4, j >> 4, RK) * 256 + (i & 15) * 16 + (j & 15)] : 0.0;
          }
#pragma unroll
        for (int y = 0; y < LB; ++y)
#pragma unroll
          for (int c = 0; c < NC; ++c) A[i0 + y][c] += v[y][c];
      }
    };
    add(std::integral_constant<int, 0>{});
    if constexpr (LB < NR) add(std::integral_constant<int, LB>{});
  } else {
#pragma unroll
    for (int ii = 0; ii < NR; ++ii)
#pragma unroll
      for (int c = 0; c < NC; ++c) {
        const int i = H * ii + h, j = lane + 64 * c;
        if (j < RP) A[ii][c] = FINAL ? P.X1[(size_t)i * RP + j] : (i == j ? 1.0 : 0.0);
      }
  }
  __syncthreads();
  // Rows kk H .. kk H + H - 1 (register row kk of each wave in turn).
  auto steps = [&](auto KK) {
    constexpr int kk = decltype(KK)::value;
    const int kend = min(H, r - kk * H);
#pragma unroll 1
    for (int hh = 0; hh < kend; ++hh) {
      const int k = kk * H + hh;
      const int buf = k & 1;
      if (h == hh) {
        if (!isE) {
          const double src = A[kk][kk * H / 64];  // row k, this lane's column of k's half
          const int lo = __builtin_amdgcn_readlane(__double2loint(src), k & 63);
          const int hi = __builtin_amdgcn_readlane(__double2hiint(src), k & 63);
          const double d = __hiloint2double(hi, lo);
          const bool ok = d > 0.0;
          const double rinv = 1.0 / d;
#pragma unroll
          for (int c = 0; c < NC; ++c) {
            const int j = lane + 64 * c;
            if (j < RP) {
              gb[buf][j] = ok ? A[kk][c] : 0.0;
              fb[buf][(j % H) * NR + j / H] = ok ? A[kk][c] * rinv : 0.0;
            }
          }
          if (lane == 0) piv[k] = ok ? d : 0.0;
        } else {
#pragma unroll
          for (int c = 0; c < NC; ++c)
            if (lane + 64 * c < RP) eb[buf][lane + 64 * c] = A[kk][c];
        }
      }
      // One barrier a step: the buffer written at step k was last read in step k - 2, before
      // the barrier of step k - 1.
      __syncthreads();
      double row[NC];
#pragma unroll
      for (int c = 0; c < NC; ++c) {
        const int j = min(lane + 64 * c, RP - 1);
        row[c] = isE ? eb[buf][j] : gb[buf][j];
      }
      const double* f = &fb[buf][h * NR];
      if (h > hh) {  // row kk H + h comes after row k
#pragma unroll
        for (int c = 0; c < NC; ++c) A[kk][c] = fma(-f[kk], row[c], A[kk][c]);
      }
#pragma unroll
      for (int ii = kk + 1; ii < NR; ++ii)
#pragma unroll
        for (int c = 0; c < NC; ++c) A[ii][c] = fma(-f[ii], row[c], A[ii][c]);
    }
  };
  static_for<0, NR>(steps);
  __syncthreads();
  if (isE) {
    double* out = FINAL ? P.M : P.X1;
#pragma unroll
    for (int ii = 0; ii < NR; ++ii) {
      const int i = H * ii + h;
      const double d = piv[i], s = d > 0.0 ? 1.0 / sqrt(d) : 0.0;
#pragma unroll
      for (int c = 0; c < NC; ++c)
        if (lane + 64 * c < RP) out[(size_t)i * RP + lane + 64 * c] = A[ii][c] * s;
    }
  }
  if (tid < RP) {
    const double rkk = sqrt(piv[tid]);
    if (!FINAL) {
      P.R1[tid] = rkk;
    } else if (tid < r) {
      const double d = rkk * P.R1[tid];
      if (P.r_diag) P.r_diag[tid] = (float)d;
      if (d == 0.0) atomicMin(&bad, tid + 1);
    }
  }
  if (FINAL) {
    __syncthreads();
    if (tid == 0 && P.info) *P.info = bad == 0x7fffffff ? 0 : bad;
  }
}

size_t part_bytes(int RK) { return (size_t)RK * (RK + 1) / 2 * 256 * 8; }

// Workspace of a panel.  The layout below (partials of 2048 rows, diag(R1), X1^T and M^T) takes less:
// the size is that of square partials per 2048 rows (r > 64: of 528 4 x 4 blocks per 1024 rows) and
// three square factors, which callers and the no-allocation variant's limit rely on.
size_t panel_ws(int rows, int RK) {
  const size_t sq = zo_align256((size_t)RK * RK * 256 * 8);
  if (RK > 4) return zo_align256((size_t)((rows + 1023) / 1024) * 528 * 16 * 8) + 3 * sq;
  return zo_align256((size_t)((rows + CHUNK - 1) / CHUNK) * RK * RK * 256 * 8) + 3 * sq;
}

// Whether the call takes short chunks of `chunk` rows, their partials in the panels' outputs: too few
// long chunks to fill the chip, every output large enough, and none over anything else that the
// call reads or writes (an Omega, another panel's output, diag(R), info).
bool short_chunks(int count, const zo_panel* panels, int r, int RK, int chunk, const int* info) {
  if (count > FEW_PANELS) return false;
  long long wg = 0;
  for (int p = 0; p < count; ++p) {
    const zo_panel& e = panels[p];
    wg += (e.rows + CHUNK - 1) / CHUNK;
    const size_t q_bytes = (size_t)e.rows * r * 4, nchunk = (size_t)((e.rows + chunk - 1) / chunk);
    if (wg >= FEW_WG || nchunk * part_bytes(RK) + 8 > q_bytes) return false;
    const uintptr_t q0 = (uintptr_t)e.q, q1 = q0 + q_bytes;
    auto over = [&](const void* a, size_t bytes) { return a && q0 < (uintptr_t)a + bytes && (uintptr_t)a < q1; };
    if (over(info, (size_t)count * 4)) return false;
    for (int o = 0; o < count; ++o) {
      const size_t bytes = (size_t)panels[o].rows * r * 4;
      if (over(panels[o].omega, bytes) || over(panels[o].r_diag, (size_t)r * 4)) return false;
      if (o != p && over(panels[o].q, bytes)) return false;
    }
  }
  return true;
}

template <int RK, int PASS>
int run_rows(const CqrArgs& ca, int wg, hipStream_t stream) {
  if (wg <= 0) return ZO_OK;
  if constexpr (RK > 4)
    hipLaunchKernelGGL((k_cqr_rows_wide<PASS>), dim3(wg), dim3(512), 0, stream, ca);
  else
    hipLaunchKernelGGL((k_cqr_rows<RK, PASS>), dim3(wg), dim3(256), 0, stream, ca);
  return zo_hip_status(hipGetLastError(), "k_cqr_rows");
}

template <int RK, bool FINAL>
int run_chol(const CqrArgs& ca, int wg, hipStream_t stream) {
  constexpr int NPAIR = RK * (RK + 1) / 2;
  const int reduced = ca.chunk != CHUNK && wg > 0;
  int st;
  if (reduced) {
    hipLaunchKernelGGL(k_cqr_reduce, dim3(NPAIR, ca.count), dim3(256), 0, stream, ca, NPAIR);
    if ((st = zo_hip_status(hipGetLastError(), "k_cqr_reduce")) != ZO_OK) return st;
  }
  hipLaunchKernelGGL((k_cqr_chol<RK, FINAL>), dim3(ca.count), dim3(RK > 4 ? 1024 : 512), 0, stream, ca, reduced);
  return zo_hip_status(hipGetLastError(), "k_cqr_chol");
}

template <int RK>
int run_batch(const CqrArgs& ca, int wg, hipStream_t stream) {
  int st;
  if ((st = run_rows<RK, 0>(ca, wg, stream)) != ZO_OK) return st;
  if ((st = run_chol<RK, false>(ca, wg, stream)) != ZO_OK) return st;
  if ((st = run_rows<RK, 1>(ca, wg, stream)) != ZO_OK) return st;
  if ((st = run_chol<RK, true>(ca, wg, stream)) != ZO_OK) return st;
  return run_rows<RK, 2>(ca, wg, stream);
}

}  // namespace

int zo_refresh_launch(int count, const zo_panel* panels, int r, int* info, void* ws,
                      size_t ws_bytes, hipStream_t stream, size_t* ws_needed) {
  const int RK = r > 64 ? WK : (r + 15) / 16;
  size_t need = zo_align256((size_t)count * sizeof(CqrPanel));
  for (int p = 0; p < count; ++p) need += panel_ws(panels[p].rows, RK);
  if (ws_needed) *ws_needed = need;
  if (!ws || count == 0) return ZO_OK;
  if (ws_bytes < need) {
    zo_set_error("refresh: workspace %zu bytes < required %zu", ws_bytes, need);
    return ZO_ERR_WORKSPACE;
  }
  const int fine = r > 64 ? WUNIT : FINE;
  const int chunk = short_chunks(count, panels, r, RK, fine, info) ? fine : CHUNK;
  WsCarver wc(ws);
  CqrPanel* tab = (CqrPanel*)wc.take((size_t)count * sizeof(CqrPanel));
  std::vector<CqrPanel> host((size_t)count);
  long long wg = 0;
  for (int p = 0; p < count; ++p) {
    CqrPanel& e = host[p];
    const int nchunk = (panels[p].rows + chunk - 1) / chunk;
    e.omega = panels[p].omega;
    e.q = panels[p].q;
    e.r_diag = panels[p].r_diag;
    e.info = info ? info + p : nullptr;
    e.part = chunk == CHUNK ? (double*)wc.take((size_t)nchunk * part_bytes(RK))
                            : (double*)(((uintptr_t)e.q + 7) & ~(uintptr_t)7);
    e.R1 = (double*)wc.take((size_t)RK * 16 * 8);
    e.X1 = (double*)wc.take((size_t)RK * RK * 256 * 8);
    e.M = (double*)wc.take((size_t)RK * RK * 256 * 8);
    e.rows = panels[p].rows;
    e.chunk_begin = (int)wg;
    wg += nchunk;
  }
  if (wg > 0x7fffffffLL) {
    zo_set_error("refresh: too many row chunks (%lld)", wg);
    return ZO_ERR_UNSUPPORTED;
  }
  int st;
  for (int c0 = 0; c0 < count; c0 += FILL_PANELS) {
    CqrFill f{};
    f.n = std::min(FILL_PANELS, count - c0);
    for (int i = 0; i < f.n; ++i) f.p[i] = host[c0 + i];
    f.dst = tab + c0;
    const int words = f.n * (int)(sizeof(CqrPanel) / 4);
    hipLaunchKernelGGL(k_cqr_fill, dim3((unsigned)((words + 255) / 256)), dim3(256), 0, stream, f);
    if ((st = zo_hip_status(hipGetLastError(), "k_cqr_fill")) != ZO_OK) return st;
  }
  CqrArgs ca{};
  ca.p = tab;
  ca.count = count;
  ca.r = r;
  ca.chunk = chunk;
  switch (RK) {
    case 1: return run_batch<1>(ca, (int)wg, stream);
    case 2: return run_batch<2>(ca, (int)wg, stream);
    case 3: return run_batch<3>(ca, (int)wg, stream);
    case 4: return run_batch<4>(ca, (int)wg, stream);
    default: return run_batch<WK>(ca, (int)wg, stream);
  }
}

// ---------------------------------------------------------------- no-allocation variant
// The scratch of zo_subspace_refresh_noalloc: a static device array, one copy per GPU the
// library runs on, held until the process ends.  The row passes write every partial Gram
// entry the Cholesky launch reads, and the Cholesky launch writes all of R1, X1 and M, so
// nothing in it has to start at zero and what an earlier call left there is never read.
// In host code the array's name is a stand-in, not a device address: the device address is
// looked up once per device (hipGetSymbolAddress, with that device current) and only that
// pointer is handed to kernels.
static __device__ __align__(256) char scratch[ZO_NOALLOC_SCRATCH_BYTES];

namespace {
constexpr int MAX_DEVICES = 64;
std::mutex g_scratch_mu;
void* g_scratch_ptr[MAX_DEVICES];
}  // namespace

int zo_refresh_scratch(void** ptr) {
  int dev = -1;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return zo_hip_status(e, "refresh_noalloc: hipGetDevice");
  if (dev < 0 || dev >= MAX_DEVICES) {
    zo_set_error("refresh_noalloc: device %d outside [0, %d)", dev, MAX_DEVICES);
    return ZO_ERR_UNSUPPORTED;
  }
  std::lock_guard<std::mutex> lock(g_scratch_mu);
  if (!g_scratch_ptr[dev]) {
    void* p = nullptr;
    e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
    if (e != hipSuccess) return zo_hip_status(e, "refresh_noalloc: hipGetSymbolAddress");
    if (!p || (uintptr_t)p % 256 != 0) {
      zo_set_error("refresh_noalloc: scratch address %p unusable", p);
      return ZO_ERR_HIP;
    }
    g_scratch_ptr[dev] = p;
  }
  *ptr = g_scratch_ptr[dev];
  return ZO_OK;
}

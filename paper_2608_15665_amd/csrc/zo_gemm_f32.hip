// fp32 GEMMs of the perturbed linear (fp32 weights and activations) on the fp32 MFMA:
//
//   Y_b = B_b A^T  (+ D_b C_b^T, the rank-r term as a second K segment)  (+ base), epilogue
//
// v_mfma_f32_16x16x4_f32 multiplies and accumulates in fp32 at 256 FLOP per clock and CU, twice
// the plain vector FMA (157 TFLOP/s at 2.4 GHz; torch's fp32 matmul reaches 153 here).  A 16-byte fragment
// (lane l: row l % 16, floats 4 (l / 16) .. + 3 of a 16-deep slice) feeds four MFMAs, element e
// of every lane in MFMA e: each MFMA takes the slice's k = 4 g + e for its four lane groups g, the
// same for both operands, so the slice's sixteen terms are each summed once.
//
// Two kernels:
//   k_f32_tile   BM x BN tiles staged through LDS, 4 waves of BM/2 x BN/2.  For calls with enough
//                tiles to fill the chip.
//   k_f32_split  16 TM x 16 TN tiles, no staging: the four waves split K (32-deep slices dealt in
//                turn), each reading its fragments straight from memory, and their sums are added
//                in wave order through LDS.  For calls with few tiles (a serial K chain on a few
//                CUs otherwise) and for the narrow projection X V.  With FAN it goes on to form
//                every block of a shared X from the tile of X W^T it holds.
// Measured (before: one 64 x 64 tile kernel on the vector FMA, K in tiles of 16 staged a float at
// a time): 8 blocks of 512 x 2048 x 2048, r = 16: 899 -> 287 us for the whole call (the product
// 703 -> 270 us, 127 TFLOP/s); the projection of the same call 212 -> 12 us; 64 x 256 x 512 with
// one X for 8 blocks 131 -> 17 us.
// Operands need only be 4-byte aligned and K may be anything: rows are read 16 bytes at a time
// (4-byte alignment is enough for the hardware's 16-byte loads), the last K % 4 floats of a row
// one by one, so nothing past a row's end is read for the last row.  Rows past the operand's end
// read its last row and are not stored.
#include "zo_internal.h"

#include <algorithm>

namespace {

typedef float f32x4_a4 __attribute__((ext_vector_type(4), aligned(4)));

__device__ __forceinline__ f32x4 mfma_f32(float a, float b, f32x4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
}

// Floats k .. k + 3 of a row of K floats (zeros from K on).
__device__ __forceinline__ f32x4 row4(const float* __restrict__ row, int k, int K) {
  if (k + 4 <= K) return (f32x4)*(const f32x4_a4*)(row + k);
  f32x4 v = {0.f, 0.f, 0.f, 0.f};
  if (k < K) v[0] = row[k];
  if (k + 1 < K) v[1] = row[k + 1];
  if (k + 2 < K) v[2] = row[k + 2];
  return v;
}

// base (if any), the epilogue and the store of four adjacent columns of one token.
__device__ __forceinline__ void finish_f32(const F32Args& a, float* Y, const float* R, int tok, int col,
                                           f32x4 v) {
  const size_t idx = (size_t)tok * a.ldy + col;
  auto one = [&](float x, size_t i) {
    if (a.base) x += a.base[i];
    if (a.epi == ZO_EPI_RELU) x = fmaxf(x, 0.f);
    if (a.epi == ZO_EPI_RESIDUAL) x += R[i];
    if (a.epi == ZO_EPI_SILU_MUL) x *= zo_silu(R[i]);
    return x;
  };
  if (col + 4 <= a.rows_a) {
    f32x4 o;
#pragma unroll
    for (int e = 0; e < 4; ++e) o[e] = one(v[e], idx + e);
    *(f32x4_a4*)(Y + idx) = (f32x4_a4)o;
  } else {
#pragma unroll
    for (int e = 0; e < 4; ++e)
      if (col + e < a.rows_a) Y[idx + e] = one(v[e], idx + e);
  }
}

// ---------------------------------------------------------------- staged tiles
// K in tiles of 32 floats (128-byte LDS rows, 16-byte chunk c of row r at c ^ ((r >> 1) & 7):
// the fragment reads of 16 consecutive rows at one chunk are conflict free), double buffered, the
// next tile's loads in registers while the current one is multiplied.  A 128 x 128 tile spends
// 4096 matrix cycles per wave on each 32 KB of loads, so it is bound by the MFMAs.
template <int BM, int BN>
__global__ __launch_bounds__(256, 2) void k_f32_tile(F32Args a) {
  constexpr int TM = BM / 32, TN = BN / 32;        // 16-row groups per wave (2 x 2 waves)
  constexpr int CA = BM / 32, CB = BN / 32;        // 16-byte chunks per thread per tile
  __shared__ __attribute__((aligned(16))) float lds[2 * (BM + BN) * 32];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wm = wave & 1, wn = wave >> 1;
  // Each XCD gets a contiguous range of tiles, grouped 8 token tiles deep, so the tiles it runs
  // at once share their operands' rows in its L2.
  const int w = blockIdx.x, nt = a.total_tiles;
  const int xcd = w & 7, widx = w >> 3;
  const int lt = xcd * (nt >> 3) + min(xcd, nt & 7) + widx;
  constexpr int GROUP = 8;
  const int nbt = a.nblk * a.tiles_b;
  const int per_group = GROUP * a.tiles_a, grp = lt / per_group, first = grp * GROUP;
  const int gsize = min(GROUP, nbt - first), rem = lt - grp * per_group;
  const int bt = first + rem % gsize;
  const int blk = bt / a.tiles_b;
  const int t0 = (bt % a.tiles_b) * BN, m0 = (rem / gsize) * BM;

  const float* __restrict__ A = a.A;
  const float* __restrict__ B = a.B + (long long)blk * a.b_block_stride;
  const float* __restrict__ C = a.ca + (long long)blk * a.ca_block_stride;
  const float* __restrict__ D = a.cb + (long long)blk * a.cb_block_stride;
  const int ntm = (a.K + 31) / 32, ntt = ntm + (a.rc + 31) / 32;
  const int lrow = tid >> 3, kc = tid & 7;  // this thread's chunk of rows lrow + 32 i
  const int pc = (kc ^ ((lrow >> 1) & 7)) * 4;
  f32x4 ra[CA], rb[CB];
  auto load = [&](int t) {
    const bool m = t < ntm;
    const float* pa = m ? A : C;
    const float* pb = m ? B : D;
    const int K = m ? a.K : a.rc, k = (m ? t : t - ntm) * 32 + kc * 4;
    if (k - kc * 4 + 32 <= K) {  // a whole tile (uniform): no per-lane check of the row's end
#pragma unroll
      for (int i = 0; i < CA; ++i)
        ra[i] = (f32x4)*(const f32x4_a4*)(pa + (size_t)min(m0 + lrow + 32 * i, a.rows_a - 1) * K + k);
#pragma unroll
      for (int i = 0; i < CB; ++i)
        rb[i] = (f32x4)*(const f32x4_a4*)(pb + (size_t)min(t0 + lrow + 32 * i, a.rows_b - 1) * K + k);
      return;
    }
#pragma unroll
    for (int i = 0; i < CA; ++i) ra[i] = row4(pa + (size_t)min(m0 + lrow + 32 * i, a.rows_a - 1) * K, k, K);
#pragma unroll
    for (int i = 0; i < CB; ++i) rb[i] = row4(pb + (size_t)min(t0 + lrow + 32 * i, a.rows_b - 1) * K, k, K);
  };
  auto store = [&](int buf) {
    float* la = lds + buf * (BM + BN) * 32;
    float* lb = la + BM * 32;
#pragma unroll
    for (int i = 0; i < CA; ++i) *(f32x4*)(la + (lrow + 32 * i) * 32 + pc) = ra[i];
#pragma unroll
    for (int i = 0; i < CB; ++i) *(f32x4*)(lb + (lrow + 32 * i) * 32 + pc) = rb[i];
  };
  f32x4 acc[TM][TN];
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j) acc[i][j] = (f32x4){0.f, 0.f, 0.f, 0.f};
  const int fr = lane & 15, fq = lane >> 4, ff = (fr >> 1) & 7;
  auto compute = [&](int buf) {
    const float* la = lds + buf * (BM + BN) * 32 + (wm * (BM / 2) + fr) * 32;
    const float* lb = lds + buf * (BM + BN) * 32 + BM * 32 + (wn * (BN / 2) + fr) * 32;
#pragma unroll
    for (int s = 0; s < 2; ++s) {
      const int ch = ((4 * s + fq) ^ ff) * 4;
      f32x4 fa[TM], fb[TN];
#pragma unroll
      for (int i = 0; i < TM; ++i) fa[i] = *(const f32x4*)(la + i * 16 * 32 + ch);
#pragma unroll
      for (int j = 0; j < TN; ++j) fb[j] = *(const f32x4*)(lb + j * 16 * 32 + ch);
#pragma unroll
      for (int e = 0; e < 4; ++e)
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
          for (int j = 0; j < TN; ++j) acc[i][j] = mfma_f32(fa[i][e], fb[j][e], acc[i][j]);
    }
  };
  if (ntt > 0) {
    load(0);
    store(0);
    __syncthreads();
    for (int t = 0; t < ntt; ++t) {
      if (t + 1 < ntt) load(t + 1);
      compute(t & 1);
      if (t + 1 < ntt) store((t + 1) & 1);
      __syncthreads();
    }
  }
  float* Y = a.Y + (long long)blk * a.y_block_stride;
  const float* R = a.R + (long long)blk * a.r_block_stride;
#pragma unroll
  for (int j = 0; j < TN; ++j) {
    const int tok = t0 + wn * (BN / 2) + 16 * j + fr;
    if (tok >= a.rows_b) continue;
#pragma unroll
    for (int i = 0; i < TM; ++i) {
      const int col = m0 + wm * (BM / 2) + 16 * i + 4 * fq;
      if (col < a.rows_a) finish_f32(a, Y, R, tok, col, acc[i][j]);
    }
  }
}

// ---------------------------------------------------------------- K split over the waves
// FAN: B is one X for every block.  The tile of X W^T, summed over the waves, stays in LDS as the
// base, and the waves of the tile's workgroups (grid z) then deal the blocks out: the rank-r term from
// zero, plus the base.
template <int TM, int TN, bool FAN>
__global__ __launch_bounds__(256) void k_f32_split(F32Args a) {
  constexpr int BM = 16 * TM, BN = 16 * TN;
  constexpr int NP = TM * TN;
  __shared__ __attribute__((aligned(16))) f32x4 red[4][NP * 64];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int fr = lane & 15, fq = lane >> 4;
  const int m0 = blockIdx.x * BM, t0 = blockIdx.y * BN, blk = FAN ? 0 : blockIdx.z;
  const float* __restrict__ A = a.A;
  const float* __restrict__ B = a.B + (long long)blk * a.b_block_stride;
  const float* __restrict__ C = a.ca + (long long)blk * a.ca_block_stride;
  const float* __restrict__ D = a.cb + (long long)blk * a.cb_block_stride;
  int rowa[TM], rowb[TN];
#pragma unroll
  for (int i = 0; i < TM; ++i) rowa[i] = min(m0 + 16 * i + fr, a.rows_a - 1);
#pragma unroll
  for (int j = 0; j < TN; ++j) rowb[j] = min(t0 + 16 * j + fr, a.rows_b - 1);
  f32x4 acc[TM][TN];
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j) acc[i][j] = (f32x4){0.f, 0.f, 0.f, 0.f};
  // 32-deep slices: the main segment's, then (not FAN) the rank segment's; wave w takes w, w + 4, ...
  const int nsm = (a.K + 31) / 32, ns = nsm + (FAN ? 0 : (a.rc + 31) / 32);
  struct Slice {
    f32x4 fa[2][TM], fb[2][TN];
  };
  auto load = [&](Slice& s, int t) {
    const bool m = t < nsm;
    const float* pa = m ? A : C;
    const float* pb = m ? B : D;
    const int K = m ? a.K : a.rc, k = (m ? t : t - nsm) * 32 + 4 * fq;
    if (k - 4 * fq + 32 <= K) {  // a whole slice (uniform)
#pragma unroll
      for (int h = 0; h < 2; ++h) {
#pragma unroll
        for (int i = 0; i < TM; ++i)
          s.fa[h][i] = (f32x4)*(const f32x4_a4*)(pa + (size_t)rowa[i] * K + k + 16 * h);
#pragma unroll
        for (int j = 0; j < TN; ++j)
          s.fb[h][j] = (f32x4)*(const f32x4_a4*)(pb + (size_t)rowb[j] * K + k + 16 * h);
      }
      return;
    }
#pragma unroll
    for (int h = 0; h < 2; ++h) {
#pragma unroll
      for (int i = 0; i < TM; ++i) s.fa[h][i] = row4(pa + (size_t)rowa[i] * K, k + 16 * h, K);
#pragma unroll
      for (int j = 0; j < TN; ++j) s.fb[h][j] = row4(pb + (size_t)rowb[j] * K, k + 16 * h, K);
    }
  };
  auto mul = [&](const Slice& s) {
#pragma unroll
    for (int h = 0; h < 2; ++h)
#pragma unroll
      for (int e = 0; e < 4; ++e)
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
          for (int j = 0; j < TN; ++j) acc[i][j] = mfma_f32(s.fa[h][i][e], s.fb[h][j][e], acc[i][j]);
  };
  // Two slices in flight ahead of the one being multiplied.
  Slice s0, s1, s2;
  int t = wave;
  if (t < ns) load(s0, t);
  if (t + 4 < ns) load(s1, t + 4);
  for (; t < ns; t += 12) {
    if (t + 8 < ns) load(s2, t + 8);
    mul(s0);
    if (t + 4 >= ns) break;
    if (t + 12 < ns) load(s0, t + 12);
    mul(s1);
    if (t + 8 >= ns) break;
    if (t + 16 < ns) load(s1, t + 16);
    mul(s2);
  }
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j) red[wave][(i * TN + j) * 64 + lane] = acc[i][j];
  __syncthreads();
  if constexpr (!FAN) {
    float* Y = a.Y + (long long)blk * a.y_block_stride;
    const float* R = a.R + (long long)blk * a.r_block_stride;
    for (int x = tid; x < NP * 64; x += 256) {
      const f32x4 v = ((red[0][x] + red[1][x]) + red[2][x]) + red[3][x];
      const int p = x >> 6, l = x & 63;
      const int tok = t0 + 16 * (p % TN) + (l & 15), col = m0 + 16 * (p / TN) + 4 * (l >> 4);
      if (tok < a.rows_b && col < a.rows_a) finish_f32(a, Y, R, tok, col, v);
    }
  } else {
    f32x4 base[TM][TN];
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
      for (int j = 0; j < TN; ++j) {
        const int x = (i * TN + j) * 64 + lane;
        base[i][j] = ((red[0][x] + red[1][x]) + red[2][x]) + red[3][x];
      }
    for (int b = __builtin_amdgcn_readfirstlane(blockIdx.z + gridDim.z * wave); b < a.fan; b += 4 * gridDim.z) {
      const float* __restrict__ Cb = a.ca + (long long)b * a.ca_block_stride;
      f32x4 d[TM][TN];
#pragma unroll
      for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j) d[i][j] = (f32x4){0.f, 0.f, 0.f, 0.f};
      for (int k = 0; k < a.rc; k += 16) {  // rc is a multiple of 16
        f32x4 fa[TM], fb[TN];
#pragma unroll
        for (int i = 0; i < TM; ++i) fa[i] = *(const f32x4*)(Cb + (size_t)rowa[i] * a.rc + k + 4 * fq);
#pragma unroll
        for (int j = 0; j < TN; ++j) fb[j] = *(const f32x4*)(a.cb + (size_t)rowb[j] * a.rc + k + 4 * fq);
#pragma unroll
        for (int e = 0; e < 4; ++e)
#pragma unroll
          for (int i = 0; i < TM; ++i)
#pragma unroll
            for (int j = 0; j < TN; ++j) d[i][j] = mfma_f32(fa[i][e], fb[j][e], d[i][j]);
      }
      float* Y = a.Y + (long long)b * a.y_block_stride;
      const float* R = a.R + (long long)b * a.r_block_stride;
#pragma unroll
      for (int j = 0; j < TN; ++j) {
        const int tok = t0 + 16 * j + fr;
        if (tok >= a.rows_b) continue;
#pragma unroll
        for (int i = 0; i < TM; ++i) {
          const int col = m0 + 16 * i + 4 * fq;
          if (col < a.rows_a) finish_f32(a, Y, R, tok, col, base[i][j] + d[i][j]);
        }
      }
    }
  }
}

template <int BM, int BN>
int launch_tile(F32Args a, hipStream_t stream) {
  a.tiles_a = (a.rows_a + BM - 1) / BM;
  a.tiles_b = (a.rows_b + BN - 1) / BN;
  const long long total = (long long)a.tiles_a * a.tiles_b * a.nblk;
  if (total > 0x7fffffffLL) {
    zo_set_error("perturbed linear: too many tiles (%lld)", total);
    return ZO_ERR_UNSUPPORTED;
  }
  a.total_tiles = (int)total;
  hipLaunchKernelGGL((k_f32_tile<BM, BN>), dim3((unsigned)total), dim3(256), 0, stream, a);
  return zo_hip_status(hipGetLastError(), "k_f32_tile");
}

// wgs: workgroups per tile (FAN).
template <int TM, int TN, bool FAN>
int launch_split(const F32Args& a, hipStream_t stream, int wgs = 1) {
  const dim3 grid((a.rows_a + 16 * TM - 1) / (16 * TM), (a.rows_b + 16 * TN - 1) / (16 * TN),
                  FAN ? wgs : a.nblk);
  hipLaunchKernelGGL((k_f32_split<TM, TN, FAN>), grid, dim3(256), 0, stream, a);
  return zo_hip_status(hipGetLastError(), "k_f32_split");
}

long long tiles(const F32Args& a, int side) {
  return (long long)((a.rows_a + side - 1) / side) * ((a.rows_b + side - 1) / side) * a.nblk;
}

// Grid limits of k_f32_split: 65535 in y and z.
bool split_fits(const F32Args& a, int tn) { return (a.rows_b + 16 * tn - 1) / (16 * tn) <= 65535 && a.nblk <= 65535; }

}  // namespace

// Staged tiles as soon as they fill the chip: 192 tiles of 128 x 128 take 3/4 of the CUs at the
// best rate per CU; 256 tiles of 64 x 64 one workgroup on each.  Below that a staged tile is a
// serial K chain on part of the chip (4 x 16 tiles of 64 x 64, 4096 deep: 870 us on the previous
// kernel, 95 us split over waves and 32 x 32 tiles).
int zo_gemm_f32(const F32Args& a, hipStream_t stream) {
  if (a.rows_a <= 0 || a.rows_b <= 0 || a.nblk <= 0) return ZO_OK;
  if (tiles(a, 128) >= 192) return launch_tile<128, 128>(a, stream);
  if (tiles(a, 64) >= 256 || !split_fits(a, 2)) return launch_tile<64, 64>(a, stream);
  return launch_split<2, 2, false>(a, stream);
}

// The projection's 16 to 128 columns: 16 tokens per workgroup, so 4096 tokens are 256 workgroups,
// the whole width in one tile up to 64 columns (X is then read once from memory).
int zo_gemm_f32_narrow(const F32Args& a, hipStream_t stream) {
  if (a.rows_a <= 0 || a.rows_b <= 0 || a.nblk <= 0) return ZO_OK;
  if (!split_fits(a, 1)) return launch_tile<64, 64>(a, stream);
  if (a.rows_a <= 16) return launch_split<1, 1, false>(a, stream);
  if (a.rows_a <= 32) return launch_split<2, 1, false>(a, stream);
  return launch_split<4, 1, false>(a, stream);
}

bool zo_gemm_f32_fans(const F32Args& a) { return tiles(a, 64) < 256; }

// Workgroups per tile: one per four blocks, a block for each wave, while the tiles leave CUs idle.  Each
// forms X W^T anew, which costs nothing on an idle CU and counts on a busy one.  Whole call, us, one /
// up to 256 workgroups in all (512 in all: the last but one 52, the last 61):
//   64 x 256 x 512, r = 4: 8 blocks 18.5 / 17.1, 128 blocks 78 / 27;   1 x 256 x 512, 256: 105 / 31
//   256 x 1024 x 2048, r = 16: 8 blocks 38.4 / 38.6, 32 blocks 51.5 / 51.2
// (Every block in full on a copied X: 17.1, 68 and 96; 101 and 293.  The smallest call's apply alone is
// 8.5 against 8.1, 9.9 with one workgroup per tile; at r = 128 the whole call 46.3 against 42.0.)
int zo_gemm_f32_fan(const F32Args& a, hipStream_t stream) {
  const long long t = (long long)((a.rows_a + 31) / 32) * ((a.rows_b + 31) / 32);
  const long long wgs = std::max(1LL, std::min(256 / t, (a.fan + 3LL) / 4));
  return launch_split<2, 2, true>(a, stream, (int)wgs);
}

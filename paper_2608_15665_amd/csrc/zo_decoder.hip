// The network a SubZero+ query evaluates (the forward inside Eq. 5 / the query
// loop of Alg. 3), as a pre-LN decoder layer of the OPT family whose six weight
// matrices are all perturbed in their own subspaces (Eq. 4):
//   A = LN1(H);  Q, K, V = A Wq'^T, A Wk'^T, A Wv'^T;  C = causal attention;
//   H2 = H + C Wo'^T;  F = relu(LN2(H2) W1'^T);  H3 = H2 + F W2'^T.
// The six products are the perturbed linears of zo_gemm.hip (the ReLU and the
// residual additions fused into their epilogues); this file adds the row
// normalisation, the attention, and the host sequence of one layer.
//
// k_layernorm: one wave per row, three passes over the row (sum, squared
// deviations, output; RMS normalisation skips the first), statistics in fp32
// with fixed-order wave sums.  Rows of
// up to 8192 elements are read once into registers (k_layernorm_reg, NC
// 512-element chunks, every load in flight at once); longer rows are re-read
// by each pass from L1/L2 (k_layernorm).  Both do the same operations in the
// same order, so their results are identical.
//
// k_attention<F16, DH, ONE>: one workgroup of 4 waves per (block, sequence, head, tile
// of 128 queries); keys in tiles of 64 through LDS (both K and V stored
// row-major), online softmax in fp32.  Each wave owns AT_NG = 2 groups of 16
// queries that share every K and V fragment it reads from LDS, skips the
// tiles whose keys all follow its queries, and computes the transposed
// products, which keeps every step in registers:
//   S^T = K Q^T  (v_mfma_f32_16x16x32: A = K rows from LDS, B = the wave's Q
//                 rows held in registers); lane (l16, g) of a 16 x 16 result
//                 holds query l16 and keys 4g .. 4g+3, so a query's softmax
//                 statistics are a sum over its lane and the 4 lanes l16 + 16g;
//   O^T += V^T P^T, 32 keys per MFMA.  The MFMA's k slots of lane group g are
//                 given the keys that lane already holds for P (4g .. 4g+3 of
//                 each of two 16-key tiles); V^T's fragment takes the same keys
//                 from two transposed reads (ds_read_b64_tr_b16) of the
//                 row-major V tile.  A sum over k does not depend on how the k
//                 slots are assigned to keys, as long as both operands use the
//                 same assignment.
// P enters as a hi + lo pair of 16-bit values (two MFMAs), so the product is
// ~2^-16 accurate before the output's rounding; P is computed as
// 2^(s scale - m + 12) (the common factor cancels in the normalisation and keeps
// fp16 low parts out of the subnormal range), with the running maximum m, a
// whole number in log2 units (a raw logit where those get coarse), moved only
// when a logit exceeds it by more than 3.
//
// What bounds it: a wave's tile is a chain (S, maximum, exponentials, conversion, P V) of about 1500
// matrix and 1600 vector cycles, and two or three waves per SIMD do not hide it.  So tile n + 1's S
// MFMAs run under tile n's first exponentials and half of P V under the rest (K double buffered),
// nothing but the last tile of a wave is masked, and 4-wave workgroups run out of step with
// each other.  The workgroups of one K/V (query tiles, grouped heads) run on one XCD.
// Before (8 waves in step, no overlap, K/V fetched per query tile) and now:
//   OPT-13B layer, 16 x 8192 x 40 x 128, 512 keys: 2325 -> 2083 us (331 TFLOP/s of visible pairs)
//   8 x 4096 x 32 x 128, 256 keys: 277 -> 268;  ... x 64: 155 -> 140
//   fp16, 8 x 8192 x 20 x 64, 2048 keys: 1406 -> 725;  4 x 8192 x 20 (4 KV) x 128, 1024 keys: 525 -> 397
#include "zo_internal.h"

#include <type_traits>

namespace {

// ---------------------------------------------------------------- layer norm
template <int DT>
__device__ __forceinline__ void load8(const void* X, size_t idx, float* v) {
  if constexpr (DT == ZO_F32) {
    const f32x4 a = *(const f32x4*)((const float*)X + idx);
    const f32x4 b = *(const f32x4*)((const float*)X + idx + 4);
    v[0] = a[0]; v[1] = a[1]; v[2] = a[2]; v[3] = a[3];
    v[4] = b[0]; v[5] = b[1]; v[6] = b[2]; v[7] = b[3];
  } else {
    const u32x4 u = *(const u32x4*)((const uint16_t*)X + idx);
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      if constexpr (DT == ZO_BF16) {
        v[2 * e] = bf16_to_f32((bf16_t)u[e]);
        v[2 * e + 1] = bf16_to_f32((bf16_t)(u[e] >> 16));
      } else {
        v[2 * e] = f16_to_f32((uint16_t)u[e]);
        v[2 * e + 1] = f16_to_f32((uint16_t)(u[e] >> 16));
      }
    }
  }
}

template <int DT>
__device__ __forceinline__ void store8(void* Y, size_t idx, const float* v) {
  if constexpr (DT == ZO_F32) {
    *(f32x4*)((float*)Y + idx) = (f32x4){v[0], v[1], v[2], v[3]};
    *(f32x4*)((float*)Y + idx + 4) = (f32x4){v[4], v[5], v[6], v[7]};
  } else if constexpr (DT == ZO_BF16) {
    *(u32x4*)((uint16_t*)Y + idx) = (u32x4){pack_bf16x2(v[0], v[1]), pack_bf16x2(v[2], v[3]),
                                            pack_bf16x2(v[4], v[5]), pack_bf16x2(v[6], v[7])};
  } else {
    *(u32x4*)((uint16_t*)Y + idx) = (u32x4){pack_f16x2(v[0], v[1]), pack_f16x2(v[2], v[3]),
                                            pack_f16x2(v[4], v[5]), pack_f16x2(v[6], v[7])};
  }
}

__device__ __forceinline__ float wave_sum(float v) {
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off, 64);
  return v;
}

// Rows of d elements (d % 8 == 0), 4 rows per workgroup, one per wave.  RMS: no centring
// (the mean is taken as 0 and the sum pass skipped) and no beta (fmaf with 0 is the rounded
// product), i.e. x / sqrt(mean(x^2) + eps) * gamma.
template <int DT, bool RMS>
__global__ __launch_bounds__(256) void k_layernorm(const void* __restrict__ X,
                                                   const float* __restrict__ gamma,
                                                   const float* __restrict__ beta, void* Y,
                                                   long long rows, int d, float eps_ln) {
  const long long row = (long long)blockIdx.x * 4 + (threadIdx.x >> 6);
  if (row >= rows) return;
  const int lane = threadIdx.x & 63;
  const size_t base = (size_t)row * d;
  float v[8];
  float mean = 0.f;
  if constexpr (!RMS) {
    float s = 0.f;
    for (int c = lane * 8; c < d; c += 512) {
      load8<DT>(X, base + c, v);
#pragma unroll
      for (int e = 0; e < 8; ++e) s += v[e];
    }
    mean = wave_sum(s) / (float)d;
  }
  float q = 0.f;
  for (int c = lane * 8; c < d; c += 512) {
    load8<DT>(X, base + c, v);
#pragma unroll
    for (int e = 0; e < 8; ++e) q = fmaf(v[e] - mean, v[e] - mean, q);
  }
  const float rstd = 1.f / sqrtf(wave_sum(q) / (float)d + eps_ln);
  for (int c = lane * 8; c < d; c += 512) {
    load8<DT>(X, base + c, v);
    const f32x4 g0 = *(const f32x4*)(gamma + c), g1 = *(const f32x4*)(gamma + c + 4);
    f32x4 b0 = {0.f, 0.f, 0.f, 0.f}, b1 = {0.f, 0.f, 0.f, 0.f};
    if constexpr (!RMS) {
      b0 = *(const f32x4*)(beta + c);
      b1 = *(const f32x4*)(beta + c + 4);
    }
    const float g[8] = {g0[0], g0[1], g0[2], g0[3], g1[0], g1[1], g1[2], g1[3]};
    const float b[8] = {b0[0], b0[1], b0[2], b0[3], b1[0], b1[1], b1[2], b1[3]};
#pragma unroll
    for (int e = 0; e < 8; ++e) v[e] = fmaf((v[e] - mean) * rstd, g[e], b[e]);
    store8<DT>(Y, base + c, v);
  }
}

// Rows of d <= 512 NC elements held in registers as loaded (8 elements per lane and chunk:
// one 16-byte word for 16-bit types, two for fp32), widened to fp32 at each use (exact).
template <int DT>
struct Raw8 {
  static constexpr int W = DT == ZO_F32 ? 2 : 1;
  u32x4 w[W];
  __device__ __forceinline__ void load(const void* X, size_t idx) {
    const u32x4* p = DT == ZO_F32 ? (const u32x4*)((const float*)X + idx) : (const u32x4*)((const uint16_t*)X + idx);
#pragma unroll
    for (int i = 0; i < W; ++i) w[i] = p[i];
  }
  __device__ __forceinline__ float at(int e) const {
    if constexpr (DT == ZO_F32) return __uint_as_float(w[e >> 2][e & 3]);
    const uint32_t u = w[0][e >> 1];
    const uint16_t h = (uint16_t)((e & 1) ? (u >> 16) : u);
    if constexpr (DT == ZO_BF16) return bf16_to_f32((bf16_t)h);
    return f16_to_f32(h);
  }
};

template <int DT, int NC, bool RMS>
__global__ __launch_bounds__(256) void k_layernorm_reg(const void* __restrict__ X,
                                                       const float* __restrict__ gamma,
                                                       const float* __restrict__ beta, void* Y,
                                                       long long rows, int d, float eps_ln) {
  const long long row = (long long)blockIdx.x * 4 + (threadIdx.x >> 6);
  if (row >= rows) return;
  const int lane = threadIdx.x & 63;
  const size_t base = (size_t)row * d;
  Raw8<DT> v[NC];
#pragma unroll
  for (int k = 0; k < NC; ++k) {
    const int c = lane * 8 + 512 * k;
    if (c < d) v[k].load(X, base + c);
  }
  float mean = 0.f;
  if constexpr (!RMS) {
    float s = 0.f;
#pragma unroll
    for (int k = 0; k < NC; ++k) {
      if (lane * 8 + 512 * k < d) {
#pragma unroll
        for (int e = 0; e < 8; ++e) s += v[k].at(e);
      }
    }
    mean = wave_sum(s) / (float)d;
  }
  float q = 0.f;
#pragma unroll
  for (int k = 0; k < NC; ++k) {
    if (lane * 8 + 512 * k < d) {
#pragma unroll
      for (int e = 0; e < 8; ++e) q = fmaf(v[k].at(e) - mean, v[k].at(e) - mean, q);
    }
  }
  const float rstd = 1.f / sqrtf(wave_sum(q) / (float)d + eps_ln);
#pragma unroll
  for (int k = 0; k < NC; ++k) {
    const int c = lane * 8 + 512 * k;
    if (c < d) {
      const f32x4 g0 = *(const f32x4*)(gamma + c), g1 = *(const f32x4*)(gamma + c + 4);
      f32x4 b0 = {0.f, 0.f, 0.f, 0.f}, b1 = {0.f, 0.f, 0.f, 0.f};
      if constexpr (!RMS) {
        b0 = *(const f32x4*)(beta + c);
        b1 = *(const f32x4*)(beta + c + 4);
      }
      const float g[8] = {g0[0], g0[1], g0[2], g0[3], g1[0], g1[1], g1[2], g1[3]};
      const float b[8] = {b0[0], b0[1], b0[2], b0[3], b1[0], b1[1], b1[2], b1[3]};
      float o[8];
#pragma unroll
      for (int e = 0; e < 8; ++e) o[e] = fmaf((v[k].at(e) - mean) * rstd, g[e], b[e]);
      store8<DT>(Y, base + c, o);
    }
  }
}

// Rotary positions, in place.  A thread owns 8 dimensions i of the first half of one head
// (and their partners dh/2 further on) in ROPE_RB consecutive rows.  The frequency
// 2^(i k), k = -2 log2(base) / dh, is formed once per thread in fp64; each angle p 2^(i k)
// is formed and reduced to [-pi, pi] in fp64, so that sincosf sees an argument that is
// exact to fp32 rounding at any position (a direct fp32 product p * theta would carry an
// absolute error of about p * 2^-24 radians: 2.4e-4 at p = 4095, a quarter of a bf16 ulp).
constexpr int ROPE_RB = 8;

template <int DT>
__global__ __launch_bounds__(256) void k_rope(void* X, long long rows, int seq_len, int d, int dh, double k) {
  const int cpr = d / 16;   // (head, 8-dimension chunk) pairs per row
  const int cph = dh / 16;  // chunks per half head
  const long long t = (long long)blockIdx.x * 256 + threadIdx.x;
  const long long groups = (rows + ROPE_RB - 1) / ROPE_RB;
  if (t >= groups * cpr) return;
  const int cc = (int)(t % cpr);
  const int h = cc / cph, c = cc % cph;
  const long long r0 = (t / cpr) * ROPE_RB;
  const long long r1 = r0 + ROPE_RB < rows ? r0 + ROPE_RB : rows;
  double theta[8];
#pragma unroll
  for (int e = 0; e < 8; ++e) theta[e] = exp2((double)(8 * c + e) * k);
  constexpr double kTwoPi = 6.283185307179586, kInvTwoPi = 0.15915494309189535;
  for (long long row = r0; row < r1; ++row) {
    const double pos = (double)(row % seq_len);
    const size_t ia = (size_t)row * d + (size_t)h * dh + 8 * c, ib = ia + dh / 2;
    float a[8], b[8], na[8], nb[8];
    load8<DT>(X, ia, a);
    load8<DT>(X, ib, b);
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      const double ang = pos * theta[e];
      const float red = (float)fma(-rint(ang * kInvTwoPi), kTwoPi, ang);
      float sn, cs;
      sincosf(red, &sn, &cs);
      na[e] = a[e] * cs - b[e] * sn;
      nb[e] = b[e] * cs + a[e] * sn;
    }
    store8<DT>(X, ia, na);
    store8<DT>(X, ib, nb);
  }
}

// ---------------------------------------------------------------- attention
constexpr int AT_NG = 2;               // 16-query groups per wave
// Waves per workgroup.  Four: two workgroups (three at 64 dims) per CU then run out of step, and one's
// exponentials cover another's MFMAs and barriers.  Eight waves that share a K/V tile were 1 to 2.2
// times slower (10 x 777 keys x 20 heads of 64, 12 blocks: 1010 against 521 us).
constexpr int AT_W = 4;
constexpr int AT_K = 64;               // keys per tile

struct AttnArgs {
  const void* Q;
  const void* K;
  const void* V;
  void* O;
  int T, seq_len, d, heads, qtiles;  // qtiles = ceil(seq_len / queries per workgroup)
  int dkv, group;                    // K/V row length (kv_heads dh); query heads per K/V head
  float scale_log2;                  // log2(e) / sqrt(dh)
};

template <bool F16>
__device__ __forceinline__ f32x4 mfma16(bf16x8 a, bf16x8 b, f32x4 c) {
  if constexpr (F16)
    return __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(f16x8, a),
                                                   __builtin_bit_cast(f16x8, b), c, 0, 0, 0);
  else
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0);
}

// Two fp32 values rounded to nearest even into a packed pair of 16-bit values (one
// v_cvt_pk_bf16_f32 / v_cvt_pk_f16_f32), and back.
typedef float f32x2_t __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x2_t __attribute__((ext_vector_type(2)));
typedef _Float16 f16x2_t __attribute__((ext_vector_type(2)));
template <bool F16>
__device__ __forceinline__ uint32_t cvt_pk(float x, float y) {
  if constexpr (F16)
    return __builtin_bit_cast(uint32_t, __builtin_convertvector((f32x2_t){x, y}, f16x2_t));
  else
    return __builtin_bit_cast(uint32_t, __builtin_convertvector((f32x2_t){x, y}, bf16x2_t));
}
template <bool F16>
__device__ __forceinline__ float unpk(uint32_t pk, int half) {
  const uint16_t h = (uint16_t)(half ? pk >> 16 : pk);
  if constexpr (F16)
    return f16_to_f32(h);
  else
    return bf16_to_f32(h);
}

typedef short i16x4_t __attribute__((ext_vector_type(4)));
// ds_read_b64_tr_b16: within each 16-lane group, lane i reads 4 consecutive 16-bit values
// D[i][0..3] at its own address, and lane j receives D[j/4 + 4e][j%4] for e = 0..3.  With
// lane i addressing row (r0 + i/4), columns c0 + 4 (i%4) of a row-major tile, lane j thus
// receives column c0 + j of rows r0 .. r0+3: a transposed fragment.
__device__ __forceinline__ u32x2 ds_read_tr(const uint16_t* p) {
  const i16x4_t v = __builtin_amdgcn_ds_read_tr16_b64_v4i16(
      (__attribute__((address_space(3))) i16x4_t*)(p));
  return __builtin_bit_cast(u32x2, v);
}

// The maximum over the four 16-lane groups.
__device__ __forceinline__ float max_groups(float x) {
  const uint32_t u = __float_as_uint(x);
  const auto a = __builtin_amdgcn_permlane16_swap(u, u, false, false);
  const uint32_t v = __float_as_uint(fmaxf(__uint_as_float(a[0]), __uint_as_float(a[1])));
  const auto b = __builtin_amdgcn_permlane32_swap(v, v, false, false);
  return fmaxf(__uint_as_float(b[0]), __uint_as_float(b[1]));
}

// Whether a running maximum m is a whole number in log2 units (see k_attention's softmax).  The scale is
// at most log2(e) / 8, so a raw logit that stands for 2^22 log2 units or more is not below 2^22 itself.
constexpr float AT_WHOLE = 4194304.f;
__device__ __forceinline__ bool at_whole(float m) { return fabsf(m) < AT_WHOLE; }

// ONE: sequences of at most one tile of keys.
template <bool F16, int DH, bool ONE>
__global__ __launch_bounds__(64 * AT_W, DH == 64 ? 3 : 2) void k_attention(AttnArgs a) {
  constexpr int W = AT_W, NT = 64 * W;  // waves, threads
  constexpr int AT_Q = 16 * AT_NG * W;  // queries per workgroup
  constexpr int KS = DH / 32;         // 32-deep k steps of Q K^T
  constexpr int DT = DH / 16;         // 16-dim tiles of the output
  constexpr int KROW = DH + 8;        // LDS row of the K tile (elements), padded
  constexpr int VROW = DH + 16;       // LDS row of the V tile (elements): 16 rows of a
                                      // transposed read fall on distinct banks
  constexpr int C8 = DH / 8;          // 16-byte chunks per head row
  constexpr int KCH = AT_K * C8 / NT;    // K (and V) chunks per thread per tile
  static_assert(KCH * NT == AT_K * C8, "tile / thread mismatch");
  __shared__ __attribute__((aligned(16))) uint16_t Ks[ONE ? 1 : 2][AT_K * KROW];
  __shared__ __attribute__((aligned(16))) uint16_t Vs[AT_K * VROW];

  // Workgroup -> (block, sequence, head, query tile).  The hardware deals workgroup w to XCD w % 8;
  // each XCD gets a contiguous range, so the query tiles (and grouped query heads) that read the same
  // K and V run on one XCD and share its L2.
  int w = (int)(blockIdx.x & 7) * (int)(gridDim.x >> 3) + min((int)(blockIdx.x & 7), (int)(gridDim.x & 7)) +
          (int)(blockIdx.x >> 3);
  const int qt = w % a.qtiles;
  w /= a.qtiles;
  const int head = w % a.heads;
  w /= a.heads;
  const int nseq = a.T / a.seq_len;
  const int seq = w % nseq;
  const int blk = w / nseq;
  const long long row0 = (long long)blk * a.T + (long long)seq * a.seq_len;  // first row of the sequence
  const int col0 = head * DH;
  const int col0kv = (head / a.group) * DH;  // the key/value head of this query head
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int l16 = lane & 15, g = lane >> 4;
  const int q0 = qt * AT_Q;  // first query of the tile (within the sequence)
  const uint16_t* __restrict__ Kg = (const uint16_t*)a.K;
  const uint16_t* __restrict__ Vg = (const uint16_t*)a.V;

  // This lane's queries (one per group) and their rows as B operands of S^T = K Q^T.
  int myq[AT_NG];
  bf16x8 qf[AT_NG][KS];
#pragma unroll
  for (int gq = 0; gq < AT_NG; ++gq) {
    myq[gq] = q0 + wave * 16 * AT_NG + 16 * gq + l16;
    const int qc = min(myq[gq], a.seq_len - 1);
    const uint16_t* qp = (const uint16_t*)a.Q + (size_t)(row0 + qc) * a.d + col0 + 8 * g;
#pragma unroll
    for (int kk = 0; kk < KS; ++kk)
      qf[gq][kk] = __builtin_bit_cast(bf16x8, *(const u32x4*)(qp + 32 * kk));
  }
  const int wq0 = q0 + wave * 16 * AT_NG;  // the wave's first query

  f32x4 o[AT_NG][DT];
  float mrow[AT_NG], lsum[AT_NG];
#pragma unroll
  for (int gq = 0; gq < AT_NG; ++gq) {
#pragma unroll
    for (int t = 0; t < DT; ++t) o[gq][t] = (f32x4){0.f, 0.f, 0.f, 0.f};
    mrow[gq] = -1e30f;  // running maximum of the logits (at_whole: in log2 units, else raw)
    lsum[gq] = 0.f;     // this lane's part of the running sum
  }

  // K and V tiles go through registers: chunk x = tid + NT c is key x / C8, dims 8 (x % C8); both are
  // stored row-major (V is read transposed by ds_read_tr).  Rows past the sequence are clamped to its
  // last row (their keys are masked).
  u32x4 kreg[KCH], vreg[KCH];
  auto load_tile = [&](const uint16_t* __restrict__ src, int k0, u32x4* reg) {
#pragma unroll
    for (int c = 0; c < KCH; ++c) {
      const int x = tid + NT * c;
      reg[c] = *(const u32x4*)(src + (size_t)(row0 + min(k0 + x / C8, a.seq_len - 1)) * a.dkv + col0kv + 8 * (x % C8));
    }
  };
  auto store_tile = [&](uint16_t* dst, int pitch, const u32x4* reg) {
#pragma unroll
    for (int c = 0; c < KCH; ++c) {
      const int x = tid + NT * c;
      *(u32x4*)&dst[(x / C8) * pitch + 8 * (x % C8)] = reg[c];
    }
  };

  // S^T of key subtile t (16 keys) from a staged K tile: st[gq][t][i] = key 16 t + 4 g + i, query
  // myq[gq].
  auto qk = [&](const uint16_t* ks, int t, f32x4 (*st)[4]) {
#pragma unroll
    for (int gq = 0; gq < AT_NG; ++gq) st[gq][t] = (f32x4){0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int kk = 0; kk < KS; ++kk) {
      const bf16x8 kf = *(const bf16x8*)&ks[(16 * t + l16) * KROW + 32 * kk + 8 * g];
#pragma unroll
      for (int gq = 0; gq < AT_NG; ++gq) st[gq][t] = mfma16<F16>(kf, qf[gq][kk], st[gq][t]);
    }
  };
  f32x4 sa[AT_NG][4];  // S^T of the tile at hand
  int raw = 0;  // whether the wave has a running maximum that is a raw logit
  // One tile of the wave: softmax and P V of st's tile.  NEXT: also the next tile's S^T (into sn, from
  // kn).  Its MFMAs have no part in this tile's chain (maximum, exponentials, conversion, P V), so
  // they run under the first half's exponentials, and the first half's P V under the second half's.
  // A tile with a successor lies wholly before the wave's queries (both are multiples of 32); the
  // last one is masked (MASK).
  auto tile = [&](auto NEXT, int k0, const uint16_t* kn, f32x4 (*st)[4], f32x4 (*sn)[4]) {
    constexpr bool next = decltype(NEXT)::value;
    // Online softmax: P = 2^(s scale - m + 12) as hi + lo 16-bit pairs in the B-operand order of the
    // P V MFMA.  m is a whole number below AT_WHOLE, so 12 - m and the rescale factor 2^(m - m') are
    // exact and each exponent is one fused multiply-add.  From there on, where s scale and m would be
    // rounded apart (from 2^26 by whole powers of two), a row's m is the raw logit and its exponent
    // (s - m) scale + 12, whose difference is exact near the maximum: P is 2^12 there at any magnitude.
    // m moves only when some query of the wave has a logit more than 3 (log2 units) above it, so most
    // tiles skip the rescale of O; P then stays at or below 2^15 (within fp16's range), and the first
    // tile sets m to its row maximum (a whole one rounded up).  OPT-13B layer: 2083 us; 2229 with
    // raw maxima alone; 2048 with whole ones alone, which cannot hold such logits.
    float cadd[AT_NG];
#pragma unroll
    for (int gq = 0; gq < AT_NG; ++gq) {
      float tmax = -1e30f;
#pragma unroll
      for (int t = 0; t < 4; ++t)
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          if (!next && k0 + 16 * t + 4 * g + i > myq[gq]) st[gq][t][i] = -INFINITY;
          tmax = fmaxf(tmax, st[gq][t][i]);
        }
      tmax = max_groups(tmax);
      const float m = mrow[gq];
      float over = fmaf(tmax, a.scale_log2, -m);
      if (__builtin_expect(raw, 0) && !at_whole(m)) over = (tmax - m) * a.scale_log2;
      if (__builtin_expect(__ballot(over > 3.f) != 0, 0)) {
        float mnew = m;
        if (over > 0.f) {
          mnew = ceilf(tmax * a.scale_log2);
          if (!at_whole(mnew)) mnew = tmax;
        }
        const float alpha = __builtin_amdgcn_exp2f(
            fmaf((at_whole(m) ? 0.f : m) - (at_whole(mnew) ? 0.f : mnew), a.scale_log2,
                 (at_whole(m) ? m : 0.f) - (at_whole(mnew) ? mnew : 0.f)));
        mrow[gq] = mnew;
        raw |= __ballot(!at_whole(mnew)) != 0;
        lsum[gq] *= alpha;
#pragma unroll
        for (int t = 0; t < DT; ++t) o[gq][t] *= alpha;
      }
      cadd[gq] = 12.f - mrow[gq];
    }
    if (__builtin_expect(raw, 0)) {
#pragma unroll
      for (int gq = 0; gq < AT_NG; ++gq)
        if (!at_whole(mrow[gq])) {
          cadd[gq] = 12.f;
#pragma unroll
          for (int t = 0; t < 4; ++t) st[gq][t] -= mrow[gq];
        }
    }
    // P of 32-key chunk c (subtiles 2 c and 2 c + 1), as the two B operands per query group.
    bf16x8 bh[2][AT_NG], bl[2][AT_NG];
    auto probs = [&](int c) {
#pragma unroll
      for (int gq = 0; gq < AT_NG; ++gq) {
        u32x4 hp, lp;
#pragma unroll
        for (int x = 0; x < 4; ++x) {
          const int t = 2 * c + (x >> 1), i = 2 * (x & 1);
          const float p0 = __builtin_amdgcn_exp2f(fmaf(st[gq][t][i], a.scale_log2, cadd[gq]));
          const float p1 = __builtin_amdgcn_exp2f(fmaf(st[gq][t][i + 1], a.scale_log2, cadd[gq]));
          lsum[gq] += p0 + p1;
          const uint32_t h = cvt_pk<F16>(p0, p1);
          hp[x] = h;
          lp[x] = cvt_pk<F16>(p0 - unpk<F16>(h, 0), p1 - unpk<F16>(h, 1));
        }
        bh[c][gq] = __builtin_bit_cast(bf16x8, hp);
        bl[c][gq] = __builtin_bit_cast(bf16x8, lp);
      }
    };
    // O^T += V^T P^T over chunk c: lane group g's k slots are keys 32 c + 4 g + (0..3) and
    // 32 c + 16 + 4 g + (0..3); V^T's fragment (dim 16 t + l16 of those keys) comes from two
    // transposed reads of the row-major V tile.
    auto pv = [&](int c) {
      const uint16_t* vb = &Vs[(32 * c + 4 * g + (l16 >> 2)) * VROW + 4 * (l16 & 3)];
#pragma unroll
      for (int t = 0; t < DT; ++t) {
        const u32x2 v0 = ds_read_tr(vb + 16 * t), v1 = ds_read_tr(vb + 16 * VROW + 16 * t);
        const bf16x8 af = __builtin_bit_cast(bf16x8, (u32x4){v0[0], v0[1], v1[0], v1[1]});
#pragma unroll
        for (int gq = 0; gq < AT_NG; ++gq) {
          o[gq][t] = mfma16<F16>(af, bh[c][gq], o[gq][t]);
          o[gq][t] = mfma16<F16>(af, bl[c][gq], o[gq][t]);
        }
      }
    };
    __builtin_amdgcn_sched_barrier(0);
    if constexpr (next) {
#pragma unroll
      for (int t = 0; t < 4; ++t) qk(kn, t, sn);
    }
    probs(0);
    if constexpr (next) {
#pragma unroll
      for (int x = 0; x < 4 * KS; ++x) {
        __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);     // a K fragment
        __builtin_amdgcn_sched_group_barrier(0x008, AT_NG, 0);  // its MFMAs
        __builtin_amdgcn_sched_group_barrier(0x002, 8 * 4 / KS, 0);
      }
    }
    __builtin_amdgcn_sched_barrier(0);
    pv(0);
    probs(1);
#pragma unroll
    for (int x = 0; x < DT; ++x) {
      __builtin_amdgcn_sched_group_barrier(0x100, 2, 1);         // a V fragment
      __builtin_amdgcn_sched_group_barrier(0x008, 2 * AT_NG, 1);  // its MFMAs
      __builtin_amdgcn_sched_group_barrier(0x002, 16 * 8 / DT, 1);
    }
    __builtin_amdgcn_sched_barrier(0);
    pv(1);
  };

  if constexpr (ONE) {
    // No next tile: nothing is staged ahead and the rows are stored from the registers, so one barrier
    // and half the registers do (94 to 143: three to five waves per SIMD), where the loop below makes
    // such calls wait on its barriers.  4 x 2048 x 20 x 128, us, before the loop / loop / this: 16 keys
    // 91 / 103 / 42, 48 keys 41.8 / 43.4 / 29.7, 64 keys 37.2 / 34.8 / 31.2.
    load_tile(Kg, 0, kreg);
    load_tile(Vg, 0, vreg);
    store_tile(Ks[0], KROW, kreg);
    store_tile(Vs, VROW, vreg);
    __syncthreads();
    if (wq0 >= a.seq_len) return;
#pragma unroll
    for (int t = 0; t < 4; ++t) qk(Ks[0], t, sa);
    tile(std::false_type{}, 0, Ks[0], sa, sa);
#pragma unroll
    for (int gq = 0; gq < AT_NG; ++gq) {
      float l = lsum[gq] + __shfl_xor(lsum[gq], 16, 64);
      l += __shfl_xor(l, 32, 64);
      if (myq[gq] >= a.seq_len) continue;
      const float inv = 1.f / l;
      uint16_t* op = (uint16_t*)a.O + (size_t)(row0 + myq[gq]) * a.d + col0 + 4 * g;
#pragma unroll
      for (int t = 0; t < DT; ++t) {
        const float y0 = o[gq][t][0] * inv, y1 = o[gq][t][1] * inv;
        const float y2 = o[gq][t][2] * inv, y3 = o[gq][t][3] * inv;
        *(u32x2*)(op + 16 * t) = F16 ? (u32x2){pack_f16x2(y0, y1), pack_f16x2(y2, y3)}
                                     : (u32x2){pack_bf16x2(y0, y1), pack_bf16x2(y2, y3)};
      }
    }
    return;
  } else {
    const int kend = min(a.seq_len, q0 + AT_Q);  // keys beyond the tile's last query are never seen
    load_tile(Kg, 0, kreg);
    store_tile(Ks[0], KROW, kreg);
    load_tile(Vg, 0, vreg);
    if (AT_K < kend) load_tile(Kg, AT_K, kreg);
    __syncthreads();
#pragma unroll
    for (int t = 0; t < 4; ++t) qk(Ks[0], t, sa);
    const int klast = min(wq0 + 16 * AT_NG, kend);  // the wave's tiles start below this
    for (int k0 = 0, n = 0; k0 < kend; k0 += AT_K, ++n) {
      // V(n) and K(n + 1) to LDS; K(n + 2) and V(n + 1) on their way.
      uint16_t* const kn = Ks[(n + 1) & 1];
      if (n) __syncthreads();  // tile n - 1 has been consumed
      store_tile(Vs, VROW, vreg);
      if (k0 + AT_K < kend) store_tile(kn, KROW, kreg);
      __syncthreads();
      if (k0 + AT_K < kend) load_tile(Vg, k0 + AT_K, vreg);
      if (k0 + 2 * AT_K < kend) load_tile(Kg, k0 + 2 * AT_K, kreg);
      if (k0 >= klast) continue;  // every key of the tile is after the wave's queries
      if (k0 + AT_K < klast) {
        f32x4 sn[AT_NG][4];
        tile(std::true_type{}, k0, kn, sa, sn);
#pragma unroll
        for (int gq = 0; gq < AT_NG; ++gq)
#pragma unroll
          for (int t = 0; t < 4; ++t) sa[gq][t] = sn[gq][t];
      } else {
        tile(std::false_type{}, k0, kn, sa, sa);
      }
    }
    // Normalise by the row sums (over the 4 lane groups).  Rows go through LDS (the K buffers, no longer
    // needed) so that a store covers whole 2 DH-byte rows instead of 16 pieces of 32 bytes.
    __syncthreads();
    uint16_t* const ow = Ks[0] + wave * 16 * AT_NG * KROW;
    static_assert(16 * AT_NG * W * KROW <= 2 * AT_K * KROW, "the staged rows fit the K buffers");
#pragma unroll
    for (int gq = 0; gq < AT_NG; ++gq) {
      float l = lsum[gq] + __shfl_xor(lsum[gq], 16, 64);
      l += __shfl_xor(l, 32, 64);
      const float inv = 1.f / l;
#pragma unroll
      for (int t = 0; t < DT; ++t) {
        const float y0 = o[gq][t][0] * inv, y1 = o[gq][t][1] * inv;
        const float y2 = o[gq][t][2] * inv, y3 = o[gq][t][3] * inv;
        const u32x2 pk = F16 ? (u32x2){pack_f16x2(y0, y1), pack_f16x2(y2, y3)}
                             : (u32x2){pack_bf16x2(y0, y1), pack_bf16x2(y2, y3)};
        *(u32x2*)&ow[(16 * gq + l16) * KROW + 16 * t + 4 * g] = pk;
      }
    }
    // Each wave reads back only its own rows.
#pragma unroll
    for (int x = lane; x < 16 * AT_NG * C8; x += 64) {
      const int row = x / C8, c = x % C8;
      const u32x4 v = *(const u32x4*)&ow[row * KROW + 8 * c];
      if (wq0 + row < a.seq_len)
        *(u32x4*)((uint16_t*)a.O + (size_t)(row0 + wq0 + row) * a.d + col0 + 8 * c) = v;
    }
  }
}

// Register-resident rows in buckets of 2, 4, 8, 10 or 16 chunks of 512; longer rows re-read.
template <int DT, bool RMS>
void layernorm_dispatch(dim3 grid, dim3 block, hipStream_t stream, const void* X, const float* gamma,
                        const float* beta, void* Y, long long rows, int d, float eps_ln) {
  if (d <= 1024)
    hipLaunchKernelGGL((k_layernorm_reg<DT, 2, RMS>), grid, block, 0, stream, X, gamma, beta, Y, rows, d, eps_ln);
  else if (d <= 2048)
    hipLaunchKernelGGL((k_layernorm_reg<DT, 4, RMS>), grid, block, 0, stream, X, gamma, beta, Y, rows, d, eps_ln);
  else if (d <= 4096)
    hipLaunchKernelGGL((k_layernorm_reg<DT, 8, RMS>), grid, block, 0, stream, X, gamma, beta, Y, rows, d, eps_ln);
  else if (d <= 5120)
    hipLaunchKernelGGL((k_layernorm_reg<DT, 10, RMS>), grid, block, 0, stream, X, gamma, beta, Y, rows, d, eps_ln);
  else if (d <= 8192)
    hipLaunchKernelGGL((k_layernorm_reg<DT, 16, RMS>), grid, block, 0, stream, X, gamma, beta, Y, rows, d, eps_ln);
  else
    hipLaunchKernelGGL((k_layernorm<DT, RMS>), grid, block, 0, stream, X, gamma, beta, Y, rows, d, eps_ln);
}

template <int DT>
void layernorm_dispatch_rms(bool rms, dim3 grid, dim3 block, hipStream_t stream, const void* X,
                            const float* gamma, const float* beta, void* Y, long long rows, int d,
                            float eps_ln) {
  if (rms)
    layernorm_dispatch<DT, true>(grid, block, stream, X, gamma, beta, Y, rows, d, eps_ln);
  else
    layernorm_dispatch<DT, false>(grid, block, stream, X, gamma, beta, Y, rows, d, eps_ln);
}

}  // namespace

int zo_layernorm_launch(long long rows, int d, int dtype, const void* X, const float* gamma,
                        const float* beta, float eps_ln, void* Y, hipStream_t stream, bool rms) {
  if (rows <= 0) return ZO_OK;
  const dim3 grid((unsigned)((rows + 3) / 4)), block(256);
  if (dtype == ZO_BF16)
    layernorm_dispatch_rms<ZO_BF16>(rms, grid, block, stream, X, gamma, beta, Y, rows, d, eps_ln);
  else if (dtype == ZO_F16)
    layernorm_dispatch_rms<ZO_F16>(rms, grid, block, stream, X, gamma, beta, Y, rows, d, eps_ln);
  else
    layernorm_dispatch_rms<ZO_F32>(rms, grid, block, stream, X, gamma, beta, Y, rows, d, eps_ln);
  return zo_hip_status(hipGetLastError(), "k_layernorm");
}

int zo_rope_launch(long long rows, int seq_len, int d, int heads, int dtype, void* X, float base,
                   hipStream_t stream) {
  const int dh = d / heads;
  const long long threads = (rows + ROPE_RB - 1) / ROPE_RB * (d / 16);
  if (threads <= 0) return ZO_OK;
  const long long wg = (threads + 255) / 256;
  if (wg > 0x7fffffffLL) {
    zo_set_error("rope: too many rows (%lld)", rows);
    return ZO_ERR_UNSUPPORTED;
  }
  const double k = -2.0 * log2((double)base) / (double)dh;
  if (dtype == ZO_BF16)
    hipLaunchKernelGGL(k_rope<ZO_BF16>, dim3((unsigned)wg), dim3(256), 0, stream, X, rows, seq_len, d, dh, k);
  else
    hipLaunchKernelGGL(k_rope<ZO_F16>, dim3((unsigned)wg), dim3(256), 0, stream, X, rows, seq_len, d, dh, k);
  return zo_hip_status(hipGetLastError(), "k_rope");
}

int zo_attention_launch(int nblk, int T, int seq_len, int d, int heads, int kv_heads, int dtype,
                        const void* Q, const void* K, const void* V, void* O, hipStream_t stream) {
  AttnArgs a;
  a.Q = Q;
  a.K = K;
  a.V = V;
  a.O = O;
  a.T = T;
  a.seq_len = seq_len;
  a.d = d;
  a.heads = heads;
  a.dkv = d / heads * kv_heads;
  a.group = heads / kv_heads;
  const int qpw = 16 * AT_NG * AT_W;
  a.qtiles = (seq_len + qpw - 1) / qpw;
  const int dh = d / heads;
  a.scale_log2 = 1.4426950408889634f / sqrtf((float)dh);
  const long long wg = (long long)nblk * (T / seq_len) * heads * a.qtiles;
  if (wg <= 0) return ZO_OK;
  if (wg > 0x7fffffffLL) {
    zo_set_error("attention: too many workgroups (%lld)", wg);
    return ZO_ERR_UNSUPPORTED;
  }
  const dim3 grid((unsigned)wg), block(64 * AT_W);
  const bool f16 = dtype == ZO_F16;
#define ZO_ATTN(F, D)                                                                            \
  if (seq_len <= AT_K) hipLaunchKernelGGL((k_attention<F, D, true>), grid, block, 0, stream, a); \
  else hipLaunchKernelGGL((k_attention<F, D, false>), grid, block, 0, stream, a)
  if (dh == 64) {
    if (f16) { ZO_ATTN(true, 64); } else { ZO_ATTN(false, 64); }
  } else {
    if (f16) { ZO_ATTN(true, 128); } else { ZO_ATTN(false, 128); }
  }
#undef ZO_ATTN
  return zo_hip_status(hipGetLastError(), "k_attention");
}

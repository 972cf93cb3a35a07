// LoRA scheme of SubZero+: the trainable parameters of an adapted layer are the
// two adapter factors A (r_L x n) and B (m x r_L), each perturbed in its own
// rank-r subspace (Eq. 4 and Alg. 2 applied to every trainable matrix; the
// paper's LoRA runs use r_L = 8, alpha = 16).  Query j with sign s gives
//   A' = A + s eps U_A Z_A,j V_A^T,   B' = B + s eps U_B Z_B,j V_B^T,
//   Y_b = X_b W^T + scale (X_b A'^T) B'^T          (scale = alpha / r_L).
// The adapter branch is a rank-(r_L + r) correction of the frozen-base GEMM:
//   X_b A'^T = X_b A^T + s eps (X_b V_A) (U_A Z_A,j)^T, so
//   Y_b = X_b W^T + P_b Bt_b^T  with  P_b = X_b [A^T | V_A]        (T x (r_L + r)),
//                                     Bt_b = scale [B' | s eps B' U_A Z_A,j]  (m x (r_L + r)).
// P_b depends on the activations only, so it is formed once per distinct X
// block by the same projection pass as the full-tuning path; Bt_b is tiny.  The
// fused GEMM of the full-tuning path then runs unchanged with rank r_L + r.
#include "zo_internal.h"

namespace {

constexpr int LR = 64;  // rows of Bt_b per workgroup

struct LoraArgs {
  const float *A, *VA, *B, *UB, *VB, *ZB, *UA, *ZA;
  void *Vt, *Bp;
  int m, n, rl, rs, rp, nblk, dtype, nb;  // nb: workgroups that form Bt (the rest form Vt)
  float eps, scale;
  BlkTable tab;
};

// Both prepared factors, one launch.
//
// Vt rows a < rl: A[a][:]; rows rl <= a < rl + rs: V_A[:][a - rl]; zero up to rp.
// 16-bit: hi part in rows [0, rp), low part (x - hi, rounded) in rows [rp, 2 rp);
// fp16 splits 256 x (the projection scales back exactly).
//
// Bt_b[i][a]: scale B'[i][a] for a < rl; scale s eps sum_c B'[i][c] (U_A Z_A,j)[c][a - rl]
// for rl <= a < rl + rs; zero up to rp, with B'[i][c] = B[i][c] + s eps sum_e U_B[i][e] (Z_B,j V_B^T)[e][c].
// Layouts as the full-tuning right factor: fp32 m x rp per block, 16-bit m x 3 rp per block as
// [hi | lo | hi].  A workgroup forms the two small products Z_B,j V_B^T and U_A Z_A,j and then
// LR rows of B' once, in LDS; a thread owns 8 adjacent columns of a row and writes 16 bytes at a
// time.  (An element per thread that redid those products took 28.6 us at 8 blocks x 1024 rows,
// r_L = 8, r = 4; both factors here take 10.8, 34.2 before.)  Every sum runs in the order of the definition.
__global__ __launch_bounds__(256) void k_lora_prep(LoraArgs p) {
  extern __shared__ float sm[];  // rs x rl, rl x rs, LR x rl
  const int tid = threadIdx.x, rl = p.rl, rs = p.rs, rp = p.rp;
  if ((int)blockIdx.x >= p.nb) {
    const long long idx = (long long)(blockIdx.x - p.nb) * 256 + tid;
    if (idx >= (long long)rp * p.n) return;
    const int a = (int)(idx / p.n), k = (int)(idx % p.n);
    float v = 0.f;
    if (a < rl)
      v = p.A[(size_t)a * p.n + k];
    else if (a < rl + rs)
      v = p.VA[(size_t)k * rs + (a - rl)];
    put_split(p.Vt, idx, (long long)rp * p.n, v, p.dtype);
    return;
  }
  float* const zv = sm;
  float* const uz = zv + rs * rl;
  float* const bq = uz + rl * rs;
  const int rowgroups = (p.m + LR - 1) / LR;
  const int b = blockIdx.x / rowgroups, i0 = (blockIdx.x % rowgroups) * LR;
  const int code = p.tab.code[b], j = code & 0xffff;
  const float se = (float)((code >> 16) - 1) * p.eps;
  const float* __restrict__ ZB = p.ZB + (size_t)j * rs * rs;
  const float* __restrict__ ZA = p.ZA + (size_t)j * rs * rs;
  for (int x = tid; x < rs * rl; x += 256) {
    const int e = x / rl, c = x % rl;
    float v = 0.f;
    for (int f = 0; f < rs; ++f) v = fmaf(ZB[e * rs + f], p.VB[(size_t)c * rs + f], v);
    zv[x] = v;
    const int c2 = x / rs, f2 = x % rs;
    float u = 0.f;
    for (int e2 = 0; e2 < rs; ++e2) u = fmaf(p.UA[(size_t)c2 * rs + e2], ZA[e2 * rs + f2], u);
    uz[x] = u;
  }
  __syncthreads();
  const int rows = min(LR, p.m - i0);
  for (int x = tid; x < rows * rl; x += 256) {
    const int i = i0 + x / rl, c = x % rl;
    float acc = 0.f;
    for (int e = 0; e < rs; ++e) acc = fmaf(p.UB[(size_t)i * rs + e], zv[e * rl + c], acc);
    bq[x] = fmaf(se, acc, p.B[(size_t)i * rl + c]);
  }
  __syncthreads();
  const int G = rp / 8;
  for (int x = tid; x < rows * G; x += 256) {
    const int row = x / G, a0 = (x % G) * 8;
    const float* br = bq + row * rl;
    float v[8];
#pragma unroll
    for (int y = 0; y < 8; ++y) {
      const int a = a0 + y;
      v[y] = 0.f;
      if (a < rl) {
        v[y] = p.scale * br[a];
      } else if (a < rl + rs) {
        float acc = 0.f;
        for (int c = 0; c < rl; ++c) acc = fmaf(br[c], uz[c * rs + a - rl], acc);
        v[y] = p.scale * se * acc;
      }
    }
    const long long o = (long long)b * p.m + i0 + row;
    if (p.dtype != ZO_F32) {
      u32x4 h, l;
#pragma unroll
      for (int y = 0; y < 4; ++y) {
        const float v0 = v[2 * y], v1 = v[2 * y + 1];
        h[y] = pack_bf16x2(v0, v1);
        l[y] = pack_bf16x2(v0 - bf16_to_f32(f32_to_bf16(v0)), v1 - bf16_to_f32(f32_to_bf16(v1)));
      }
      bf16_t* d = (bf16_t*)p.Bp + o * 3 * rp + a0;
      *(u32x4*)d = h;
      *(u32x4*)(d + rp) = l;
      *(u32x4*)(d + 2 * rp) = h;
    } else {
      float* d = (float*)p.Bp + o * rp + a0;
      *(f32x4*)d = (f32x4){v[0], v[1], v[2], v[3]};
      *(f32x4*)(d + 4) = (f32x4){v[4], v[5], v[6], v[7]};
    }
  }
}

}  // namespace

int zo_lora_prepare(const PlinearPlan& p, int rl, int rs, const int* blk_query,
                    const int8_t* blk_sign, float eps, float scale, const void* X, const float* A,
                    const float* UA, const float* VA, const float* ZA, const float* B,
                    const float* UB, const float* VB, const float* ZB, void* ws,
                    hipStream_t stream) {
  const PlinearWs w = zo_plinear_ws(p, ws);
  LoraArgs a{};
  a.A = A; a.VA = VA; a.B = B; a.UB = UB; a.VB = VB; a.ZB = ZB; a.UA = UA; a.ZA = ZA;
  a.Vt = w.vt;
  a.Bp = w.bp;
  a.m = p.m;
  a.n = p.n;
  a.rl = rl;
  a.rs = rs;
  a.rp = p.rp;
  a.nblk = p.nblk;
  a.dtype = p.in_dtype;
  a.eps = eps;
  a.scale = scale;
  a.tab = zo_blk_table(p.nblk, blk_query, blk_sign);
  const long long nb = (long long)p.nblk * ((p.m + LR - 1) / LR);
  const long long nv = ((long long)p.rp * p.n + 255) / 256;
  if (nb + nv > 0x7fffffffLL) {
    zo_set_error("LoRA prepare: too many workgroups (%lld)", nb + nv);
    return ZO_ERR_UNSUPPORTED;
  }
  a.nb = (int)nb;
  const size_t lds = (size_t)(2 * rs * rl + LR * rl) * sizeof(float);  // at most 51.2 KB (rl + rs <= 128)
  hipLaunchKernelGGL(k_lora_prep, dim3((unsigned)(nb + nv)), dim3(256), lds, stream, a);
  const int st = zo_hip_status(hipGetLastError(), "k_lora_prep");
  if (st != ZO_OK) return st;
  return zo_plinear_project(p, X, ws, stream);
}

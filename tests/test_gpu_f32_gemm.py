"""The fp32 perturbed linear at the sizes where its GEMM changes kernel or runs off a tile: the
waves-split kernel, the 64 and 128 staged tiles, the one-launch and two-launch shared-X forms, every
width of the projection, K and column remainders of 1 to 3 floats, and operands that are aligned to
4 bytes and no more.  Against float64 at the fp32 bar of the other tests (floored relative error at
rms 1e-5: a K-term fp32 sum carries about sqrt(K) 2^-24 relative to the rms, 3e-6 at K = 2049)."""
import numpy as np
import pytest
import torch

import paper_2608_15665_amd as zo
from _common import ferr

pytestmark = pytest.mark.gpu


def _dev(a, off):
    """a on the GPU as a contiguous tensor that starts `off` floats into its allocation."""
    flat = torch.empty(a.size + 4, dtype=torch.float32, device="cuda")
    v = flat[off:off + a.size].view(a.shape)
    v.copy_(torch.from_numpy(np.ascontiguousarray(a, dtype=np.float32)))
    return v


@pytest.mark.parametrize("T,m,n,r,q,shared,off,epi", [
    (1, 1, 1, 1, 1, False, 0, "none"),
    (17, 33, 31, 3, 2, False, 1, "none"),        # split kernel, one slice with a remainder
    (33, 30, 129, 16, 2, True, 3, "none"),       # one-launch shared X
    (40, 50, 2049, 17, 1, True, 0, "relu"),      # projection of 32 columns, K = 64 slices + 1
    (100, 70, 130, 33, 2, False, 2, "residual"),  # projection of 48 columns
    (20, 140, 67, 65, 1, True, 1, "silu"),       # 80 columns
    (17, 40, 33, 5, 3, True, 1, "residual"),     # ... 6 blocks dealt to 8 waves of a tile's two workgroups
    (100, 300, 64, 20, 9, True, 0, "none"),      # 18 blocks to 20 waves of 5 workgroups
    (300, 500, 40, 5, 10, True, 2, "relu"),      # 160 tiles: one workgroup each, 5 blocks per wave
    (260, 700, 45, 100, 4, False, 1, "none"),    # 64 x 64 tiles, projection of 112 columns
    (1500, 1030, 70, 8, 2, False, 3, "residual"),  # 128 x 128 tiles
    (1501, 1027, 34, 20, 1, True, 1, "relu"),    # shared X through the base
])
def test_f32_gemm_paths(T, m, n, r, q, shared, off, epi):
    rng = np.random.default_rng(T * 7 + m)
    nblk = 2 * q
    f = lambda *s: rng.standard_normal(s).astype(np.float32)  # noqa: E731
    X, W, Z = f(T if shared else nblk * T, n), f(m, n), f(q, r, r)
    U, V = f(m, r) / np.float32(np.sqrt(m)), f(n, r) / np.float32(np.sqrt(n))
    R = f(nblk * T, m)
    bq, bs = [b // 2 for b in range(nblk)], [1 - 2 * (b % 2) for b in range(nblk)]
    bs[-1] = 0
    p = zo.PerturbedLinear(_dev(X, off), _dev(W, off), _dev(U, off), _dev(V, off), _dev(Z, off), bq, bs, 0.5, T,
                           x_block_stride=0 if shared else T * n, Y=_dev(np.zeros((nblk * T, m)), off))
    p.prepare()
    code = {"none": zo.ZO_EPI_NONE, "relu": zo.ZO_EPI_RELU, "residual": zo.ZO_EPI_RESIDUAL,
            "silu": zo.ZO_EPI_SILU_MUL}[epi]
    Y = p.apply(code, _dev(R, off) if epi in ("residual", "silu") else None).cpu().numpy().astype(np.float64)
    d = lambda a: a.astype(np.float64)  # noqa: E731
    for b in range(nblk):
        x = d(X) if shared else d(X[b * T:(b + 1) * T])
        ref = x @ (d(W) + bs[b] * 0.5 * d(U) @ d(Z[bq[b]]) @ d(V).T).T
        rb = d(R[b * T:(b + 1) * T])
        if epi == "relu":
            ref = np.maximum(ref, 0)
        elif epi == "residual":
            ref = ref + rb
        elif epi == "silu":
            ref = ref * rb / (1 + np.exp(-rb))
        assert ferr(Y[b * T:(b + 1) * T], ref, 1.0) <= 1e-5, b

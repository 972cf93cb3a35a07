"""The shared-X fan-out at its tile edges: token and column remainders of the 128 x 128 tiles, every
rank width (32 to 128, one or two fragments of odd and even count), block counts that do and do not
split evenly over workgroups, all output types, plain and ReLU.

Each output is held to the bound its arithmetic sets: the output's rounding (half an ulp: 2^-8 of
the value for bf16, 2^-11 for fp16), 2^-15 of the rank-r term's absolute sum |X||V||U Z| (its
operands are hi + lo pairs, 2^-17 relative each, and the dropped lo lo product is below 2^-17) and
2^-20 of the absolute sum |X||W| and of the rank-r one (fp32 sums of at most 96 + 3 * 128 terms).
"""
import numpy as np
import pytest
import torch

import paper_2608_15665_amd as zo
from _common import cast, dev_f32, host, orth
import zo_draws as zd

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dt", ["bf16", "f16"])
@pytest.mark.parametrize("T,m,n,r,nblk", [
    (1, 8, 32, 1, 2),            # one token, one chunk of columns
    (127, 136, 64, 32, 3),       # a token short of a tile; 8 columns past one
    (129, 120, 96, 33, 5),       # a token past; 8 columns short; r padded to 64
    (300, 264, 64, 64, 16),      # more blocks than a tile's share of workgroups takes evenly
    (130, 392, 32, 80, 7),       # r padded to 96
    (256, 256, 64, 128, 2),      # whole tiles, widest rank
    (3000, 2056, 32, 16, 9),     # 24 x 17 tiles: several blocks per workgroup
])
def test_fan_out_edges(T, m, n, r, nblk, dt):
    q = (nblk + 1) // 2
    W, Wv = cast(zd.draw(3, "W0", (m, n), (m, n), 0.02), dt)
    X, Xv = cast(zd.draw(3, "X", (T, n, 0), (T, n)), dt)
    rr = min(r, m, n)
    U, V = orth(3, (1, m, rr), m, rr), orth(3, (2, n, rr), n, rr)
    Z = zd.z_draws(3, 0, 0, q, rr)
    bq = [b // 2 for b in range(nblk)]
    bs = [(1, -1, 0)[b % 3] for b in range(nblk)]
    out16 = torch.bfloat16 if dt == "bf16" else torch.float16
    base = Xv @ Wv.T
    P = Xv @ V.astype(np.float64)
    refs = [base + bs[b] * 0.5 * P @ (U.astype(np.float64) @ Z[bq[b]].astype(np.float64)).T for b in range(nblk)]
    Xa, Wa = np.abs(Xv), np.abs(Wv)
    bmag = Xa @ Wa.T
    rmag = [abs(bs[b]) * 0.5 * (Xa @ np.abs(V).astype(np.float64)) @ np.abs(U.astype(np.float64) @ Z[bq[b]].astype(np.float64)).T
            for b in range(nblk)]
    half_ulp = 2.0 ** -8 if dt == "bf16" else 2.0 ** -11
    for out in (out16, torch.float32):
        p = zo.PerturbedLinear(X, W, dev_f32(U), dev_f32(V), dev_f32(Z), bq, bs, 0.5, T, x_block_stride=0,
                               out_dtype=out)
        p.prepare()
        for epi in (zo.ZO_EPI_NONE, zo.ZO_EPI_RELU):
            p.Y.fill_(float("nan"))
            Y = host(p.apply(epi)).reshape(nblk, T, m)
            for b in range(nblk):
                ref = np.maximum(refs[b], 0) if epi == zo.ZO_EPI_RELU else refs[b]
                u = half_ulp if out == out16 else 2.0 ** -24
                tol = u * np.abs(ref) + 2.0 ** -15 * rmag[b] + 2.0 ** -20 * (bmag + rmag[b]) + 2.0 ** -25
                err = np.abs(Y[b] - ref)
                assert np.all(err <= tol), (b, epi, float(np.max(err / tol)))

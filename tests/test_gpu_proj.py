"""The prepare's projection at the edges of its tiles: every tile shape (64, 128 and 256 tokens; one,
two and three factors), token remainders, K a multiple of 8 that ends anywhere in a 64-deep tile.

eps = 1 and fp32 outputs put the rank-r term at the size of the output; against float64 each value
is held to 2^-15 of the rank-r term's absolute sum (hi + lo operands, 2^-17 relative each) plus 2^-20
of all absolute sums (fp32 sums of a few hundred terms)."""
import numpy as np
import pytest
import torch

import paper_2608_15665_amd as zo
from _common import cast, dev_f32, host, orth
import zo_draws as zd

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dt", ["bf16", "f16"])
@pytest.mark.parametrize("T,n,r,nblk,count", [
    (63, 8, 3, 2, 1),            # 64 tokens, one chunk of K
    (65, 72, 40, 3, 1),          # a token past a tile, 8 past a K tile, r padded to 64
    (130, 104, 30, 2, 2),        # K tail in the second half of a tile
    (200, 96, 20, 2, 3),
    (8200, 120, 16, 4, 1),       # 128-token tiles with a remainder, one factor
    (8200, 88, 33, 4, 1),        # ... of 128 rows
    (8192, 64, 17, 4, 2),
    (8200, 200, 32, 4, 3),
    (32790, 40, 50, 2, 1),       # 256-token tiles
    (32790, 136, 9, 2, 2),
    (32790, 32, 9, 2, 3),        # the main GEMM's stack
    (32790, 40, 9, 2, 3),        # the main GEMM in fp32, combined apart: a ragged stack of 192 rows
    (300, 72, 40, 2, 2),         # ... of 256 rows
])
def test_projection_tiles(T, n, r, nblk, count, dt):
    m, q = 16, nblk
    rng = np.random.default_rng(T + n)
    X, Xv = cast(rng.standard_normal((nblk * T, n)), dt)
    r = min(r, n)
    bq, bs = list(range(nblk)), [1, -1, 1, -1][:nblk]
    ops, mats = [], []
    for i in range(count):
        mi = m + 8 * i
        W, Wv = cast(zd.draw(i, "W0", (mi, n), (mi, n), 0.02), dt)
        U, V = rng.standard_normal((mi, r)).astype(np.float32) / 4, orth(i, (2, n, r), n, r)
        Z = zd.z_draws(i, 0, 0, q, r)
        need = zo.lib().zo_perturbed_linear_workspace(T, mi, n, r, q, nblk, T * n, 1)
        ops.append(zo.PerturbedLinear(X, W, dev_f32(U), dev_f32(V), dev_f32(Z), bq, bs, 1.0, T, x_block_stride=T * n,
                                      out_dtype=torch.float32,
                                      workspace=torch.empty(need, dtype=torch.uint8, device="cuda")))
        mats.append((Wv, U.astype(np.float64), V.astype(np.float64), Z.astype(np.float64)))
    if count > 1:
        zo.prepare_group(ops)
    else:
        ops[0].prepare()
    rows = np.unique(np.concatenate([np.arange(min(T, 70)), np.arange(max(0, T - 70), T), rng.integers(0, T, 200)]))
    for op, (Wv, U, V, Z) in zip(ops, mats):
        Y = host(op.apply()).reshape(nblk, T, -1)
        for b in range(nblk):
            x = Xv[b * T:(b + 1) * T][rows]
            uz = bs[b] * U @ Z[bq[b]]
            ref = x @ Wv.T + (x @ V) @ uz.T
            base, rank = np.abs(x) @ np.abs(Wv).T, np.abs(x) @ np.abs(V) @ np.abs(uz).T
            err = np.abs(Y[b][rows] - ref)
            tol = 2.0 ** -15 * rank + 2.0 ** -20 * (base + rank) + 2.0 ** -30
            assert np.all(err <= tol), (b, float(np.max(err / tol)))

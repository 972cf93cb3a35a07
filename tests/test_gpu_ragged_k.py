"""K that ends anywhere in a 64-deep tile (a multiple of 8): the main GEMM reads the columns past K as
zero.  Every remainder class (one to eight chunks, first or second half of the tile), with one to
thirteen K tiles, every output type and epilogue.

A row of X and a row of W hold NaN: their own outputs are NaN, and nothing of them may reach the
neighbouring rows, whose last tile's loads run over into them.  Bounds: half an ulp of the output
(2^-8 of the value for bf16, 2^-11 for fp16, 2^-24 for fp32), 2^-15 of the rank-r term's absolute sum
(hi + lo operands), 2^-19 of all absolute sums (fp32 sums of up to 1000 terms); the gated epilogue
carries a few fp32 ulps of silu (2^-20) on top."""
import numpy as np
import pytest
import torch

import paper_2608_15665_amd as zo
from _common import cast, dev_f32, host, orth
import zo_draws as zd

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dt", ["bf16", "f16"])
@pytest.mark.parametrize("n", [8, 24, 40, 56, 72, 136, 168, 184, 200, 264, 360, 440, 776, 808])
@pytest.mark.parametrize("epi", ["none", "relu", "residual", "silu"])
def test_ragged_k(n, epi, dt):
    T, m, r, q = 70, 264, 5, 1
    code = {"none": zo.ZO_EPI_NONE, "relu": zo.ZO_EPI_RELU, "residual": zo.ZO_EPI_RESIDUAL,
            "silu": zo.ZO_EPI_SILU_MUL}[epi]
    rng = np.random.default_rng(n)
    bad_t, bad_m = 33, 100
    X64, W64 = rng.standard_normal((2 * T, n)), rng.standard_normal((m, n)) * 0.05
    X64[bad_t] = X64[T + bad_t] = np.nan
    W64[bad_m] = np.nan
    X, W = cast(np.nan_to_num(X64), dt)[0], cast(np.nan_to_num(W64), dt)[0]
    Xv, Wv = host(X), host(W)
    X[bad_t] = X[T + bad_t] = float("nan")
    W[bad_m] = float("nan")
    U, V = rng.standard_normal((m, r)).astype(np.float32) / 4, orth(1, (2, n, r), n, r)
    Z = zd.z_draws(1, 0, 0, q, r)
    out16 = torch.bfloat16 if dt == "bf16" else torch.float16
    keep_t, keep_m = np.arange(T) != bad_t, np.arange(m) != bad_m
    for out in (out16, torch.float32):
        R = cast(rng.standard_normal((2 * T, m)), dt)[0] if out == out16 else dev_f32(rng.standard_normal((2 * T, m)))
        Rv = host(R)
        op = zo.PerturbedLinear(X, W, dev_f32(U), dev_f32(V), dev_f32(Z), [0, 0], [1, -1], 0.5, T, x_block_stride=T * n,
                                out_dtype=out)
        op.prepare()
        Y = host(op.apply(code, R if epi in ("residual", "silu") else None)).reshape(2, T, m)
        u = 2.0 ** -24 if out == torch.float32 else 2.0 ** -8 if dt == "bf16" else 2.0 ** -11
        for b, s in ((0, 0.5), (1, -0.5)):
            x, rb = Xv[b * T:(b + 1) * T], Rv[b * T:(b + 1) * T]
            uz = s * U.astype(np.float64) @ Z[0].astype(np.float64)
            ref = x @ Wv.T + (x @ V) @ uz.T
            rank = np.abs(x) @ np.abs(V) @ np.abs(uz).T
            tol = 2.0 ** -15 * rank + 2.0 ** -19 * (np.abs(x) @ np.abs(Wv).T + rank)
            if epi == "relu":
                ref = np.maximum(ref, 0)
            elif epi == "residual":
                ref = ref + rb
            elif epi == "silu":
                g = rb / (1 + np.exp(-rb))
                ref, tol = ref * g, tol * np.abs(g) + 2.0 ** -20 * np.abs(ref * g)
            tol = tol + u * np.abs(ref) + 2.0 ** -25
            err = np.abs(Y[b] - ref)[keep_t][:, keep_m]
            assert np.all(err <= tol[keep_t][:, keep_m]), (b, out, float(np.nanmax(err / tol[keep_t][:, keep_m])))
            if epi != "relu":
                assert np.isnan(Y[b][bad_t]).all() and np.isnan(Y[b][:, bad_m]).all()

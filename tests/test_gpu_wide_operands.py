"""Operands beyond the buffer descriptors of the main kernels (X of 2 GiB with n % 32 != 0, of 4 GiB
otherwise): the register-staged GEMM takes the product and the projection, then the separate combine.

Sampled rows against float64, each value held to half an ulp of the output (2^-8 of the value for
bf16, 2^-11 for fp16, 2^-24 for fp32), 2^-15 of the rank-r term's absolute sum (hi + lo operands)
and 2^-17 of all absolute sums (fp32 accumulators that take 16 terms at a time: 130 roundings of
2^-24 for 2056 terms); the gated epilogue carries a few fp32 ulps of silu (2^-20) on top."""
import numpy as np
import pytest
import torch

import paper_2608_15665_amd as zo
from _common import dev_f32, orth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dt", [torch.bfloat16, torch.float16])
@pytest.mark.parametrize("T,n,m,r", [
    (522256, 2056, 8, 3),       # 2 GiB + 0.5 MB: 64 factor rows, one row tile
    (522256, 2056, 264, 40),    # 128 factor rows, columns past a 256-row tile
    (522256, 2056, 16, 100),    # r > 64
    (1048584, 2048, 24, 20),    # 4 GiB + 32 KB
])
def test_spans_beyond_the_descriptors(T, n, m, r, dt):
    g = torch.Generator(device="cuda")
    g.manual_seed(T + m)
    rnd = lambda *s, dtype=dt: torch.randn(*s, generator=g, device="cuda", dtype=dtype)  # noqa: E731
    X, W = rnd(T, n), rnd(m, n) * 0.05
    assert X.numel() * 2 > (2 ** 31 if n % 32 else 2 ** 32 - 256)
    r = min(r, n)
    U, V, Z = rnd(m, r, dtype=torch.float32) / 4, dev_f32(orth(1, (2, n, r), n, r)), rnd(1, r, r, dtype=torch.float32)
    rows = torch.cat([torch.arange(300, device="cuda"), torch.arange(T - 300, T, device="cuda"),
                      torch.randint(0, T, (400,), generator=g, device="cuda")])
    x, w, v = X[rows].double(), W.double(), V.double()
    uz = 0.5 * U.double() @ Z[0].double()
    rank_abs = (x.abs() @ v.abs()) @ uz.abs().t()
    base, rank, mag = x @ w.t(), (x @ v) @ uz.t(), x.abs() @ w.abs().t() + rank_abs
    for out in (dt, torch.float32):
        op = zo.PerturbedLinear(X, W, U, V, Z, [0, 0], [1, 0], 0.5, T, x_block_stride=0, out_dtype=out)
        op.prepare()
        u = 2.0 ** -24 if out == torch.float32 else 2.0 ** -8 if dt == torch.bfloat16 else 2.0 ** -11
        for epi in (zo.ZO_EPI_NONE, zo.ZO_EPI_RELU, zo.ZO_EPI_RESIDUAL, zo.ZO_EPI_SILU_MUL):
            R = rnd(2 * T, m, dtype=out) if epi in (zo.ZO_EPI_RESIDUAL, zo.ZO_EPI_SILU_MUL) else None
            op.Y.fill_(float("nan"))
            Y = op.apply(epi, R).view(2, T, m)
            for b in range(2):
                ref, tol = (base + rank, 2.0 ** -15 * rank_abs + 2.0 ** -17 * mag) if b == 0 else (base, 2.0 ** -17 * mag)
                if epi == zo.ZO_EPI_RELU:
                    ref = ref.clamp_min(0)
                elif R is not None:
                    rb = R.view(2, T, m)[b][rows].double()
                    if epi == zo.ZO_EPI_RESIDUAL:
                        ref = ref + rb
                    else:
                        gate = rb * torch.sigmoid(rb)
                        ref, tol = ref * gate, tol * gate.abs() + 2.0 ** -20 * (ref * gate).abs()
                err = (Y[b][rows].double() - ref).abs()
                ratio = err / (tol + u * ref.abs() + 2.0 ** -25)
                assert bool((ratio <= 1).all()), (epi, b, out, float(ratio.max()))  # a NaN fails
            del Y, R
        del op
    torch.cuda.empty_cache()

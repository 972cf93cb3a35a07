"""Causal attention at the edges of its tiles (64 keys, 32 queries per wave, 128 per workgroup), with
plain and grouped heads, and with logits that keep moving the running maximum: rising along the keys
(every tile rescales), falling (none after the first), and large enough (hundreds) that P spans the
whole exponent range.  Bars: those of the attention tests."""
import numpy as np
import pytest
import torch

import paper_2608_15665_amd as zo
from _common import cast, check_attention, host

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dt", ["bf16", "f16"])
@pytest.mark.parametrize("seq", [1, 15, 16, 17, 31, 32, 33, 47, 48, 49, 63, 64, 65, 96, 127, 128, 129, 160, 193, 257, 520])
@pytest.mark.parametrize("heads,kv,dh,shape", [(2, 2, 64, "plain"), (4, 2, 128, "rise"), (3, 1, 64, "fall"),
                                               (2, 1, 128, "large")])
def test_attention_tile_edges(seq, heads, kv, dh, shape, dt):
    rng = np.random.default_rng(seq * 10 + heads)
    nblk, nseq = 2, 2
    T = nseq * seq
    Q, K, V = (rng.standard_normal((nblk * T, h * dh)) for h in (heads, kv, kv))
    pos = np.tile(np.arange(seq), nblk * nseq)[:, None]
    if shape in ("rise", "fall"):  # logits along a fixed direction grow or shrink by ~0.2 a key
        Q[:, ::dh] = 3.0
        K[:, ::dh] = (pos if shape == "rise" else seq - pos) * 0.2 * np.sqrt(dh) / 3.0
    elif shape == "large":
        Q, K = 4 * Q, 4 * K
    (Qd, Qv), (Kd, Kv), (Vd, Vv) = (cast(a, dt) for a in (Q, K, V))
    O = torch.full_like(Qd, float("nan"))
    zo.causal_attention(Qd, Kd, Vd, nblk, T, seq, heads, out=O, kv_heads=kv)
    got = host(O)
    for b in range(nblk):
        sl = slice(b * T, (b + 1) * T)
        check_attention(got[sl], Qv[sl], Kv[sl], Vv[sl], heads, seq, dt, (b, shape), kv)


@pytest.mark.parametrize("dt,c", [("f16", 506.0), ("f16", 1000.0), ("f16", 2048.0), ("f16", 2056.0), ("f16", 8192.0), ("f16", 16376.0),
                                  ("bf16", 512.0), ("bf16", 1024.0), ("bf16", 8192.0), ("bf16", 2.0 ** 20), ("bf16", 2.0 ** 45)])
@pytest.mark.parametrize("dh", [64, 128])
def test_attention_huge_logits(dh, dt, c):
    """Logits up to dh c^2 (finite in fp32), where a rounding of s scale alone is worth whole powers of
    two; the smaller c put the running maximum on both sides of 2^22, where its form changes.  Equal
    keys have equal logits, so their average is an ordinary one; otherwise the logits differ by so much
    that one key has all the weight, and the output is its row of V bit for bit."""
    rng = np.random.default_rng(dh)

    def run(q, k, v):
        seq = len(k)
        (Qd, Qv), (Kd, Kv), (Vd, Vv) = (cast(np.tile(x, (2, 1)), dt) for x in (q, k, v))
        O = torch.full_like(Qd, float("nan"))
        zo.causal_attention(Qd, Kd, Vd, 1, 2 * seq, seq, 1, out=O)
        return host(O), Qv, Kv, Vv

    for seq in (1, 2, 48, 64, 70, 200):  # all keys equal
        full = np.full((seq, dh), c)
        O, Qv, Kv, Vv = run(full, full, rng.standard_normal((seq, dh)))
        check_attention(O, Qv, Kv, Vv, 1, seq, dt, (c, seq))
        np.testing.assert_array_equal(O[::seq], Vv[::seq])  # the first query sees one key
    seq = 200
    full, v = np.full((seq, dh), c), rng.standard_normal((seq, dh))
    top = 77  # one dominant key, after which every query takes its row; before it, key 0 dominates
    k = np.full((seq, dh), c / 4)
    k[0], k[top] = c / 2, c
    O, _, _, Vv = run(full, k, v)
    want = np.where((np.arange(2 * seq) % seq < top)[:, None], Vv[0], Vv[top])
    np.testing.assert_array_equal(O, want)
    # each key above all before it (the running maximum moves in every tile): a query takes its own row
    O, _, _, Vv = run(full, full * (np.arange(1, seq + 1) / 256)[:, None], v)
    np.testing.assert_array_equal(O, Vv)
    # the same from far below zero
    O, _, _, Vv = run(full, -full * (np.arange(seq, 0, -1) / 256)[:, None], v)
    np.testing.assert_array_equal(O, Vv)
    # all logits far below zero, the first the largest
    O, _, _, Vv = run(full, -full * (np.arange(1, seq + 1) / 256)[:, None], v)
    np.testing.assert_array_equal(O, np.broadcast_to(Vv[0], Vv.shape))

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
@pytest.mark.parametrize("seq", [1, 31, 32, 33, 63, 64, 65, 96, 127, 128, 129, 160, 193, 257, 520])
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

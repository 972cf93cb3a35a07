"""The update at the edges of its tiles: 256-row workgroups and 512-column strips (r <= 64), 512 and 256
(r > 64), 64-row tiles of L, ranks that end anywhere in a 16-deep slice, factors aligned to 4 bytes.

The fp32 value before storage is held to the update's bound
E = (3 2^-18 + (3 rp + r + 4) 2^-24) (lr |U||S|)|V|^T + 2^-23 |W| (hi + lo pairs keep L and V to 2^-18 and
drop lo lo; 3 rp products and L's r terms accumulate in fp32; one rounding of W - delta); the stored
16-bit value is exactly its rounding to nearest even.  fp32 W: the same with r terms and no split."""
import numpy as np
import pytest
import torch

import oracle
import paper_2608_15665_amd as zo
from _common import cast, host, orth
import zo_draws as zd

pytestmark = pytest.mark.gpu


def _off(a, off):
    flat = torch.empty(a.size + 4, dtype=torch.float32, device="cuda")
    v = flat[off:off + a.size].view(a.shape)
    v.copy_(torch.from_numpy(np.ascontiguousarray(a, dtype=np.float32)))
    return v


@pytest.mark.parametrize("dt", ["bf16", "f16", "f32"])
@pytest.mark.parametrize("m,n,r,off", [
    (63, 8, 3, 0), (65, 504, 17, 1), (255, 512, 31, 2), (257, 520, 32, 3), (513, 1032, 33, 1), (300, 1016, 50, 2),
    (256, 248, 63, 3), (700, 136, 64, 0), (511, 264, 65, 1), (513, 256, 97, 2), (129, 520, 128, 0)])
def test_update_tile_edges(m, n, r, off, dt):
    q, lr, b1, b2, ea, t = 3, np.float32(1e-2), np.float32(0.9), np.float32(0.95), np.float32(1e-8), 4
    rng = np.random.default_rng(m + r)
    rr = min(r, m, n)
    W, Wv = cast(zd.draw(5, "W0", (m, n), (m, n), 0.02), dt)
    U, V, Z = orth(5, (1, m, rr), m, rr), orth(5, (2, n, rr), n, rr), zd.z_draws(5, 0, 0, q, rr)
    M1 = rng.standard_normal((rr, rr)).astype(np.float32) * np.float32(0.1)
    M2 = np.square(rng.standard_normal((rr, rr)).astype(np.float32) * np.float32(0.3))
    g = rng.standard_normal(q).astype(np.float32)
    wout = torch.empty((m, n), dtype=torch.float32, device="cuda")
    it = dict(W=W, U=_off(U, off), V=_off(V, off), Z=_off(Z, off), M1=_off(M1, off), M2=_off(M2, off), w_f32_out=wout)
    zo.subspace_adam_update([it], _off(g, off), t, float(lr), float(b1), float(b2), float(ea))
    d = lambda a: np.asarray(a, np.float64)  # noqa: E731
    ref = oracle.subspace_adam_update(d(Wv), d(U), d(V), d(Z), d(g), d(M1), d(M2), t, float(lr), float(b1), float(b2),
                                      float(ea))
    zb = (d(g)[:, None, None] * d(Z)).mean(0)
    m1, m2 = float(b1) * d(M1) + (1 - float(b1)) * zb, float(b2) * d(M2) + (1 - float(b2)) * zb * zb
    S = (m1 / (1 - float(b1) ** t)) / (np.sqrt(m2 / (1 - float(b2) ** t)) + float(ea))
    mag = float(lr) * (np.abs(d(U)) @ np.abs(S)) @ np.abs(d(V)).T
    rp = (rr + 31) // 32 * 32
    if dt == "f32":
        bound = (2 * rr + 4) * 2.0 ** -24 * mag + 2.0 ** -23 * np.abs(ref["W"])
    else:
        bound = (3 * 2.0 ** -18 + (3 * rp + rr + 4) * 2.0 ** -24) * mag + 2.0 ** -23 * np.abs(ref["W"])
    got = wout.cpu().numpy()
    err = np.abs(got.astype(np.float64) - ref["W"])
    assert np.all(err <= bound), float(np.max(err / bound))
    stored = {"bf16": oracle.round_bf16, "f16": oracle.round_f16, "f32": lambda x: x}[dt](got.astype(np.float64))
    np.testing.assert_array_equal(host(W), stored)


@pytest.mark.parametrize("r", [65, 96, 97, 128])
def test_update_of_many_rows(r):
    """Calls of many rows at r > 64 form 128 rows of L per workgroup: every item of one such call is
    bitwise what it is alone (64 rows per workgroup), with row counts on both sides of both tiles."""
    rng = np.random.default_rng(r)
    sizes = [(129, 40), (64, 136), (191, 8), (65600, 8), (128, 264)]
    assert sum(m for m, _ in sizes) >= 65536
    q, g = 2, _off(rng.standard_normal(2), 0)

    def items():
        gen = torch.Generator(device="cuda")
        gen.manual_seed(r)
        f = lambda *s: torch.randn(*s, generator=gen, device="cuda")  # noqa: E731
        return [dict(W=f(m, n).mul_(0.02).bfloat16(), U=f(m, r).mul_(0.1), V=f(n, r).mul_(0.1), Z=f(q, r, r),
                     M1=f(r, r).mul_(0.1), M2=f(r, r).square_()) for m, n in sizes]

    together, alone = items(), items()
    step = lambda its: zo.subspace_adam_update(its, g, 4, 1e-2, 0.9, 0.95, 1e-8)  # noqa: E731
    step(together)
    for k, (m, n) in enumerate(sizes):
        if m < 65536:
            step([alone[k]])
        else:  # its rows in two calls of fewer
            it, h = alone[k], 32896
            for sl in (slice(0, h), slice(h, m)):
                part = dict(it, W=it["W"][sl].clone(), U=it["U"][sl].clone(), M1=it["M1"].clone(), M2=it["M2"].clone())
                step([part])
                it["W"][sl] = part["W"]
            it["M1"], it["M2"] = part["M1"], part["M2"]
        for name in ("W", "M1", "M2"):
            assert torch.equal(together[k][name], alone[k][name]), (k, name)

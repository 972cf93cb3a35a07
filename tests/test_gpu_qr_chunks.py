"""The refresh's short and long row chunks, and its two row kernels (r <= 64 and r <= 128).

A panel's sums are the same tree whatever the chunk length, so its Q, diag(R) and info are the same
bits in a call of few panels (short chunks, partials in their outputs, where every output holds its
partials: SHORT; long ones in ROWS, whose smallest panels do not), in place (long chunks: the output
lies over Omega) and among enough panels to make the call take long chunks; and against a float64 Householder
QR with the sign fix at the refresh's bar (1e-5 elementwise; the factor is exact to fp32 rounding,
so 2e-7 normwise holds with room).  Rows sit on the edges of the units (128 and 256 rows), the short
chunks (512 and 256) and the long ones (2048)."""
import numpy as np
import pytest
import torch

import paper_2608_15665_amd as zo
from _common import dev_f32, normwise

pytestmark = pytest.mark.gpu

ROWS = {
    1: [1, 7, 512, 513, 2049],
    15: [15, 127, 128, 129, 4097],
    17: [511, 513, 2047, 6000],
    48: [48, 640, 2048],
    64: [64, 2050, 5120, 8191],
    65: [65, 255, 257, 2049],
    100: [128, 512, 4100],
    128: [128, 129, 2047, 2048, 8193],
}
SHORT = {  # from the fewest rows whose output holds the partials of its short chunks
    2: [257, 2049],
    15: [35, 127, 128, 129, 4097],
    17: [91, 511, 513, 2047, 6000],
    48: [65, 640, 2048, 2049],
    64: [81, 2050, 5120, 8191],
    73: [253, 2048, 5120],
    100: [185, 512, 4100],
    128: [145, 2047, 2048, 8193],
}


def _ref(om):
    Q, R = np.linalg.qr(om.astype(np.float64))
    s = np.sign(np.diag(R))
    return Q * s, np.abs(np.diag(R))


def run(om, r, out, rd=None, info=None):
    n = len(om)
    rd = [torch.empty(r, device="cuda") for _ in range(n)] if rd is None else rd
    info = torch.full((n,), -1, dtype=torch.int32, device="cuda") if info is None else info
    zo.subspace_refresh(om, r, out=out, r_diag=rd, info=info)
    return [o.cpu().numpy() for o in out], [d.cpu().numpy() for d in rd], info.cpu().numpy()


def _holds_partials(rows, r):
    chunk, tiles = (512, (r + 15) // 16) if r <= 64 else (256, 8)
    return -(-rows // chunk) * (tiles * (tiles + 1) // 2) * 2048 + 8 <= rows * r * 4


@pytest.mark.parametrize("r,sizes", sorted(ROWS.items()) + sorted(SHORT.items()))
def test_chunks_agree_bitwise_and_with_householder(r, sizes):
    assert all(_holds_partials(rows, r) for rows in sizes) == (SHORT.get(r) is sizes or r == 17)
    rng = np.random.default_rng(r)
    host = [rng.standard_normal((rows, r)).astype(np.float32) for rows in sizes]
    oms = [dev_f32(h) for h in host]

    alone, rda, infa = run(oms, r, [torch.full_like(o, float("nan")) for o in oms])
    place = [o.clone() for o in oms]
    inpl, rdi, infi = run(place, r, place)
    filler = dev_f32(rng.standard_normal((max(r, 32), r)))
    crowd = oms + [filler] * 70  # more panels than a call with short chunks holds
    many, rdm, _ = run(crowd, r, [torch.empty_like(o) for o in crowd])
    for p, h in enumerate(host):
        for q, d in ((inpl, rdi), (many, rdm)):
            np.testing.assert_array_equal(alone[p].view(np.uint32), q[p].view(np.uint32), err_msg=str(h.shape))
            np.testing.assert_array_equal(rda[p].view(np.uint32), d[p].view(np.uint32))
        if h.shape[0] >= 2 * r:
            Q, R = _ref(h)
            assert np.abs(alone[p] - Q).max() <= 1e-5 and normwise(alone[p], Q) <= 2e-7, h.shape
            assert normwise(rda[p], R) <= 2e-7
    assert not infa.any() and not infi.any()


@pytest.mark.parametrize("r,sizes", [(64, [5120, 2050, 300]), (17, [4097, 600, 511]), (128, [4100, 2048, 500])])
def test_outputs_that_overlap(r, sizes):
    """One scratch output for every panel of a call that wants diag(R) and info only, and diag(R) or info
    inside another panel's output: each value that the call leaves whole is that of separate calls."""
    rng = np.random.default_rng(r + 1)
    oms = [dev_f32(rng.standard_normal((rows, r))) for rows in sizes]
    oms[1][:, r // 2] = 0  # one rank-deficient panel, so that info differs
    ref = [run([o], r, [torch.empty_like(o)]) for o in oms]
    refq, refd, refi = ([x[k][0] for x in ref] for k in range(3))
    assert [int(i) for i in refi] == [0, r // 2 + 1, 0]
    same = lambda a, b: np.testing.assert_array_equal(a.view(np.uint32), b.view(np.uint32))  # noqa: E731

    scratch = torch.empty(max(sizes) * r, device="cuda")
    _, rd, info = run(oms, r, [scratch[:o.numel()].view(o.shape) for o in oms])
    assert list(info) == list(refi)
    for p in range(3):
        same(rd[p], refd[p])
    # A panel's rows shifted into the next one's output: only the last written is whole.
    _, rd, info = run(oms, r, [scratch[4 * p:4 * p + o.numel()].view(o.shape) for p, o in enumerate(oms)])
    assert list(info) == list(refi)
    for p in range(3):
        same(rd[p], refd[p])

    for p in range(3):  # the outputs are written last: whole, over whatever lay in them
        out = [torch.empty_like(o) for o in oms]
        rds = [torch.empty(r, device="cuda") for _ in oms]
        rds[(p + 1) % 3] = out[p].view(-1)[8:8 + r]
        q, rd, info = run(oms, r, out, rd=rds)
        assert list(info) == list(refi)
        for k in range(3):
            same(q[k], refq[k])
            if k != (p + 1) % 3:
                same(rd[k], refd[k])
        out = [torch.empty_like(o) for o in oms]
        q, rd, _ = run(oms, r, out, info=out[p].view(-1)[4:7].view(torch.int32))
        for k in range(3):
            same(q[k], refq[k])
            same(rd[k], refd[k])


@pytest.mark.parametrize("r", [16, 64, 100])
@pytest.mark.parametrize("bad", [float("nan"), float("inf")])
def test_non_finite_panel_is_reported(r, bad):
    """At the entry's column or before it, and the call's other panels are what they are alone."""
    rng = np.random.default_rng(r)
    om = [dev_f32(rng.standard_normal((600, r))) for _ in range(2)]
    alone, _, _ = run([om[1]], r, [torch.empty_like(om[1])])
    om[0][5, r - 3] = bad
    q, _, info = run(om, r, [torch.empty_like(o) for o in om])
    assert 1 <= info[0] <= r - 2 and info[1] == 0
    np.testing.assert_array_equal(q[1].view(np.uint32), alone[0].view(np.uint32))

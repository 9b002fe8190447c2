"""Sums of two points on a quad of lanes whose Y coordinate, a difference of two
separately reduced products, lies below -p.

Five copies of one point P in one bucket are cut into 2 P and 3 P, which a quad
adds; the bucket is the only one of its window, so the reduction hands the sum's
raw Y on.  The multiples k of G below were found by replaying that arithmetic in
exact integers (about one point in 10^5 on BN254, one in 10^7 on BLS12-381); the
replay stands here too."""

import numpy as np
import pytest

import synthetic as syn
from oracle import c_oracle as co
from oracle import curves, ref
from tests.common import points_to_rows, rows_to_points

BELOW = {"bn254": [10013050, 20048954, 40055868, 60040826, 70030660, 80036618], "bls12_381": [50126061, 71332620]}
RADIX = {"bn254": 261, "bls12_381": 392}
CASES = [(name, k) for name, ks in BELOW.items() for k in ks]
COPIES = 5


def merged_y(c, k):
    """Y of the quad's 2 P + 3 P for P = k G, over p, with P's lanes as in the bucket sums."""
    p, e = c.p, RADIX[c.name]
    mask = (1 << e) - 1
    pinv = (-pow(p, -1, 1 << e)) & mask

    def red(t):
        return (t + ((t * pinv) & mask) * p) >> e

    x, y = (v * (1 << e) % p for v in ref.scalar_mul(c, k, ref.generator(c)))
    u = 2 * y  # 2 P
    v = red(u * u)
    w, s, m = red(u * v), red(x * v), 3 * red(x * x)
    x2 = red(m * m) - 2 * s
    y2, z2, zz2 = red(m * (s - x2) - w * y), v, w
    d, r = red(x * z2) - x2, red(y * zz2) - y2  # + P
    pp = red(d * d)
    ppp, q = red(d * pp), red(x2 * pp)
    x3 = red(r * r) - ppp - 2 * q
    y3, z3, zz3 = red(r * (q - x3) - y2 * ppp), red(z2 * pp), red(zz2 * ppp)
    u1, s1 = red(x2 * z3), red(y2 * zz3)  # 2 P + 3 P on the quad
    d, r = red(z2 * x3) - u1, red(zz2 * y3) - s1
    pp = red(d * d)
    ppp, q = red(d * pp), red(u1 * pp)
    return (red(r * (q - (red(r * r) - ppp - 2 * q))) - red(s1 * ppp)) / p


@pytest.mark.parametrize("name,k", CASES)
def test_the_inputs_leave_the_range(name, k):
    assert -1.1 < merged_y(curves.CURVES[name], k) <= -1.0


def _copies(c, ks):
    k = syn.ints_to_limbs([k for k in ks for _ in range(COPIES)], 4)
    return co.fixed_base(c.cid, c.limbs, k)


def _ones(n):
    s = np.zeros((n, 4), dtype=np.uint64)
    s[:, 0] = 1
    return s


@pytest.mark.gpu
@pytest.mark.parametrize("name,k", CASES)
def test_one_msm(name, k):
    torch = pytest.importorskip("torch")
    eccmi = pytest.importorskip("paper_2501_03245_amd")
    c = curves.CURVES[name]
    dev = lambda a: torch.from_numpy(np.ascontiguousarray(a).view(np.int64).copy()).cuda()
    out = torch.zeros(2 * c.limbs, dtype=torch.int64, device="cuda")
    inf = torch.zeros(1, dtype=torch.uint8, device="cuda")
    with eccmi.Context(0) as ctx:
        eccmi.ecc_msm(ctx, c.cid, dev(_copies(c, [k])), dev(_ones(COPIES)), COPIES, out, inf, window_c=16)
    got = rows_to_points(c, out.cpu().numpy().view(np.uint64).reshape(1, -1), inf.cpu().numpy())
    assert got == [ref.scalar_mul(c, COPIES * k, ref.generator(c))]


# 48 MSMs at this width are more reduction waves than the quad form of the
# reduction takes; with more than 2^14 MSMs in all (the others empty) the
# windows are combined one MSM per lane, on unsigned limbs
@pytest.mark.gpu
@pytest.mark.parametrize("empty", [0, 16384])
@pytest.mark.parametrize("name", sorted(BELOW))
def test_a_batch_of_small_msms(name, empty):
    torch = pytest.importorskip("torch")
    eccmi = pytest.importorskip("paper_2501_03245_amd")
    c = curves.CURVES[name]
    m = 48
    ks = [BELOW[name][j % len(BELOW[name])] for j in range(m)]
    offs = np.concatenate([np.arange(m + 1) * COPIES, np.full(empty, m * COPIES)])
    dev = lambda a: torch.from_numpy(np.ascontiguousarray(a).view(np.int64).copy()).cuda()
    out = torch.ones((m + empty) * 2 * c.limbs, dtype=torch.int64, device="cuda")
    inf = torch.zeros(m + empty, dtype=torch.uint8, device="cuda")
    with eccmi.Context(0) as ctx:
        eccmi.ecc_msm_batch(ctx, c.cid, dev(_copies(c, ks)), dev(_ones(m * COPIES)), offs, out, inf, window_c=8)
    exp = points_to_rows(c, [ref.scalar_mul(c, COPIES * k, ref.generator(c)) for k in ks] + [None] * empty)
    np.testing.assert_array_equal(out.cpu().numpy().view(np.uint64).reshape(m + empty, -1), exp)

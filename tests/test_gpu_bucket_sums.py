"""Edges of the direct bucket sums: buckets that are cut into parts (few, many,
and more than one workgroup's lanes of them), buckets of one entry, equal and
opposite points inside a part and across parts, and empty calls, against the
discrete-log identity or the oracle, exactly."""

import numpy as np
import pytest

import synthetic as syn
from oracle import curves
from tests.common import dlog_msm_expected, rows_to_points, seeded_bases, seeded_scalars

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
eccmi = pytest.importorskip("paper_2501_03245_amd")


def msm(c, bases, s, flags=0, window_c=0):
    out = torch.zeros(2 * c.limbs, dtype=torch.int64, device="cuda")
    inf = torch.zeros(1, dtype=torch.uint8, device="cuda")
    with eccmi.Context(0) as ctx:
        eccmi.ecc_msm(ctx, c.cid, torch.from_numpy(np.ascontiguousarray(bases).view(np.int64).copy()).cuda(),
                      torch.from_numpy(np.ascontiguousarray(s).view(np.int64).copy()).cuda(), len(s), out, inf,
                      flags=flags, window_c=window_c)
        torch.cuda.synchronize()
    return rows_to_points(c, out.cpu().numpy().view(np.uint64).reshape(1, -1), inf.cpu().numpy())[0]


# one digit for every scalar: a bucket of n entries, n / 4 parts of it
@pytest.mark.parametrize("name", ["bn254", "bls12_381"])
@pytest.mark.parametrize("n", [4, 5, 17, 64, 65, 1023, 1025, 5000])
def test_one_bucket_in_many_parts(name, n):
    c = curves.CURVES[name]
    k, bases = seeded_bases(name, n, 501)
    s = np.zeros((n, 4), dtype=np.uint64)
    s[:, 0] = 3
    assert msm(c, bases, s, eccmi.ECC_NO_ENDOMORPHISM, 4) == dlog_msm_expected(c, k, s)


# the same points again, or their negatives, so that a part meets P + P and
# P - P, and whole parts and the merge meet equal and opposite sums
@pytest.mark.parametrize("name", ["bn254", "bls12_381"])
@pytest.mark.parametrize("period", [1, 2, 4, 8])
@pytest.mark.parametrize("mirror", [False, True])
def test_repeated_and_opposite_points(name, period, mirror):
    c = curves.CURVES[name]
    n = 96
    k, bases = seeded_bases(name, n, 502)
    idx = np.arange(n) % period
    k, bases = k[idx].copy(), bases[idx].copy()
    if mirror:
        for i in range(n):
            if (i // period) % 2:
                y = syn.limbs_to_int(bases[i, c.limbs:])
                bases[i, c.limbs:] = syn.ints_to_limbs([c.p - y], c.limbs)[0]
                k[i] = syn.ints_to_limbs([c.r - syn.limbs_to_int(k[i])], 4)[0]
    s = np.zeros((n, 4), dtype=np.uint64)
    s[:, 0] = 5
    for flags in (0, eccmi.ECC_NO_ENDOMORPHISM):
        assert msm(c, bases, s, flags, 5) == dlog_msm_expected(c, k, s)


@pytest.mark.parametrize("name,n,wc", [("bn254", 1, 0), ("bls12_381", 2, 0), ("bls12_381", 257, 16),
                                       ("bn254", 3000, 13), ("bls12_381", 20011, 0)])
def test_sizes_and_windows(name, n, wc):
    c = curves.CURVES[name]
    k, bases = seeded_bases(name, n, 503)
    s = seeded_scalars(name, n, 504)
    assert msm(c, bases, s, 0, wc) == dlog_msm_expected(c, k, s)
    assert msm(c, bases, np.zeros_like(s), 0, wc) is None

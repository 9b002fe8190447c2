"""Sums of cut buckets' parts: few, many and very many parts, by lanes, by quads
and by workgroups, where parts are equal, opposite or O, against the discrete-log
identity, exactly; and cuts that follow the entries that a call really has."""

import numpy as np
import pytest

import synthetic as syn
from oracle import curves
from tests.common import dlog_msm_expected, rows_to_points, seeded_bases

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
eccmi = pytest.importorskip("paper_2501_03245_amd")


def msm(c, bases, s, window_c=0):
    out = torch.zeros(2 * c.limbs, dtype=torch.int64, device="cuda")
    inf = torch.zeros(1, dtype=torch.uint8, device="cuda")
    with eccmi.Context(0) as ctx:
        ctx.set_profiling(True)
        eccmi.ecc_msm(ctx, c.cid, torch.from_numpy(np.ascontiguousarray(bases).view(np.int64).copy()).cuda(),
                      torch.from_numpy(np.ascontiguousarray(s).view(np.int64).copy()).cuda(), len(s), out, inf,
                      window_c=window_c)
        torch.cuda.synchronize()
        adds = ctx.stats()["round_adds"]
    return rows_to_points(c, out.cpu().numpy().view(np.uint64).reshape(1, -1), inf.cpu().numpy())[0], adds


# `per` copies of one point (or its negative) in each bucket, 4 entries a part:
# 3 parts of a bucket go to 1-4 lanes, 10, 38 and 75 to 16, 250 to
# workgroups.  3000 points at c = 13 are merged by lanes, 900 at c = 16 and 600
# at c = 8 by quads (the second then meets the lane form of the reduction).
@pytest.mark.parametrize("name", ["bn254", "bls12_381"])
@pytest.mark.parametrize("n,window_c", [(3000, 13), (900, 16), (600, 8)])
@pytest.mark.parametrize("per", [12, 40, 150, 300, 1000])
@pytest.mark.parametrize("mirror", [False, True])
def test_equal_and_opposite_parts(name, n, window_c, per, mirror):
    c = curves.CURVES[name]
    k, bases = seeded_bases(name, 256, 511)
    b = np.arange(n) // per
    k, bases = k[b].copy(), bases[b].copy()
    if mirror:
        for i in range(1, n, 2):
            y = syn.limbs_to_int(bases[i, c.limbs:])
            bases[i, c.limbs:] = syn.ints_to_limbs([c.p - y], c.limbs)[0]
            k[i] = syn.ints_to_limbs([c.r - syn.limbs_to_int(k[i])], 4)[0]
    s = np.zeros((n, 4), dtype=np.uint64)
    s[:, 0] = b + 1 if window_c > 8 else b % 100 + 1
    assert msm(c, bases, s, window_c)[0] == dlog_msm_expected(c, k, s)


# one bucket of so many parts that every workgroup of the widest spread adds some
@pytest.mark.parametrize("name", ["bn254", "bls12_381"])
@pytest.mark.parametrize("n", [1028, 65536, 70000, 200003])
def test_one_bucket_over_many_workgroups(name, n):
    c = curves.CURVES[name]
    k, bases = seeded_bases(name, 1000, 512)
    i = np.arange(n) % 1000
    s = np.zeros((n, 4), dtype=np.uint64)
    s[:, 0] = 1
    got, adds = msm(c, bases[i], s)
    assert got == dlog_msm_expected(c, k[i], s)
    # parts of at most 4 + n / 2^16 entries, whatever the bound on all windows' entries is
    assert adds <= n - n // (5 + n // 65536)


# a captured call whose scalars change in place: cuts, lists and counters are
# made anew on the device at every replay
@pytest.mark.parametrize("name", ["bn254", "bls12_381"])
def test_replays_follow_the_scalars(name):
    c = curves.CURVES[name]
    n = 20000
    k, bases = seeded_bases(name, 1000, 513)
    i = np.arange(n) % 1000
    uniform = syn.uniform_below(514, syn.TAG_SCALARS, n, c.r, 4)
    small = uniform & np.array([0xFF, 0, 0, 0], dtype=np.uint64)
    ones = np.zeros_like(uniform)
    ones[:, 0] = 1
    b = torch.from_numpy(np.ascontiguousarray(bases[i]).view(np.int64).copy()).cuda()
    s = torch.zeros((n, 4), dtype=torch.int64, device="cuda")
    out = torch.zeros(2 * c.limbs, dtype=torch.int64, device="cuda")
    inf = torch.zeros(1, dtype=torch.uint8, device="cuda")
    with eccmi.Context(0) as ctx:
        for values in (uniform, ones, 0 * ones, small, ones, uniform):
            s.copy_(torch.from_numpy(values.view(np.int64).copy()))
            eccmi.ecc_msm(ctx, c.cid, b, s, n, out, inf, flags=eccmi.ECC_USE_GRAPH)
            torch.cuda.synchronize()
            got = rows_to_points(c, out.cpu().numpy().view(np.uint64).reshape(1, -1), inf.cpu().numpy())[0]
            assert got == dlog_msm_expected(c, k[i], values)

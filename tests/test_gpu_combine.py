"""Special cases of the window combination and the ends of the digit walk, against
the CPU oracle, exactly: a window sum equal to the doubled running sum, its
negation, windows without points between others, and scalars whose digits carry
through every window up to the top, at widths that divide the scalar or leave a
narrow top window, alone and grouped in a batch."""

import numpy as np
import pytest

import synthetic as syn
from oracle import c_oracle as co
from oracle import curves, ref
from tests.common import points_to_rows, rows_to_points, seeded_bases, seeded_scalars

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
eccmi = pytest.importorskip("paper_2501_03245_amd")


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a).view(np.int64).copy()).cuda()


def cases(c, wc):
    """(multiples of G, scalars) of small MSMs at window width wc."""
    r, h = c.r, 1 << wc
    high = 1 << (wc * (120 // wc))
    runs = [(1 << b) - 1 for b in (wc - 1, wc, wc + 1, 127, 128, c.scalar_bits - 1)]
    halves = [sum(1 << (wc * i + wc - 1) for i in range(c.scalar_bits // wc)), r - 1, r - h, (r >> 1) + 1]
    return [
        ([1, h], [h, 1]),                        # the doubled running sum meets itself
        ([1, r - h], [h, 1]),                    # and its negation: O
        ([1, r - h, 5], [h * h, h, 3]),          # O on the way, then a point
        ([3, 7], [high, 1]),                     # windows without points between
        ([2] * len(runs), [min(v, r - 1) for v in runs]),
        (list(range(1, len(halves) + 1)), [min(v, r - 1) for v in halves]),
    ]


@pytest.mark.parametrize("name", ["bn254", "bls12_381"])
@pytest.mark.parametrize("wc", [3, 8, 11, 16])
@pytest.mark.parametrize("endo", [True, False])
def test_combination_special_cases(name, wc, endo):
    c = curves.CURVES[name]
    sets = cases(c, wc)
    flags = 0 if endo else eccmi.ECC_NO_ENDOMORPHISM
    k = [v for ks, _ in sets for v in ks]
    s = syn.ints_to_limbs([v for _, ss in sets for v in ss], 4)
    bases = co.fixed_base(c.cid, c.limbs, syn.ints_to_limbs(k, 4))
    offs = np.cumsum([0] + [len(ks) for ks, _ in sets]).astype(np.uint64)
    want = []
    for ks, ss in sets:
        e = sum(a * b for a, b in zip(ks, ss)) % c.r
        want.append(ref.scalar_mul(c, e, ref.generator(c)) if e else None)
    m = len(sets)
    bd, sd = dev(bases), dev(s)
    got = []
    with eccmi.Context(0) as ctx:
        for i in range(m):
            lo, hi = int(offs[i]), int(offs[i + 1])
            out = torch.full((2 * c.limbs,), -1, dtype=torch.int64, device="cuda")
            inf = torch.full((1,), 255, dtype=torch.uint8, device="cuda")
            eccmi.ecc_msm(ctx, c.cid, bd[lo:hi].contiguous(), sd[lo:hi].contiguous(), hi - lo, out, inf,
                          flags=flags, window_c=wc)
            torch.cuda.synchronize()
            got += rows_to_points(c, out.cpu().numpy().view(np.uint64).reshape(1, -1), inf.cpu().numpy())
        outs = torch.full((m * 2 * c.limbs,), -1, dtype=torch.int64, device="cuda")
        infs = torch.full((m,), 255, dtype=torch.uint8, device="cuda")
        eccmi.ecc_msm_batch(ctx, c.cid, bd, sd, offs, outs, infs, flags=flags, window_c=wc)
        torch.cuda.synchronize()
        batch = rows_to_points(c, outs.cpu().numpy().view(np.uint64).reshape(m, -1), infs.cpu().numpy())
    assert points_to_rows(c, got).tolist() == points_to_rows(c, want).tolist()
    assert points_to_rows(c, batch).tolist() == points_to_rows(c, want).tolist()


@pytest.mark.parametrize("endo", [True, False])
@pytest.mark.parametrize("wc", [0, 2, 13])
def test_batch_grouping_split_edges(endo, wc):
    """MSMs whose windows are grouped by one workgroup and those that share
    them (more than 2048 grouped points, a point counting twice with the
    endomorphism split), with fewer windows than workgroups' shares are even
    (W = 10 or 20 at c = 13) and with points at infinity."""
    c = curves.BLS12_381
    at = 1024 if endo else 2048
    sizes = [at, at + 1, 0, 1, at - 1, 3 * at + 5]
    offs = np.cumsum([0] + sizes).astype(np.uint64)
    n = int(offs[-1])
    _, bases = seeded_bases(c.name, n, 931)
    bases = bases.copy()
    bases[::97] = 0
    s = seeded_scalars(c.name, n, 932, kind="bits")
    out, inf = co.msm_batch(c.cid, c.limbs, bases, s, offs)
    m = len(sizes)
    outs = torch.full((m * 2 * c.limbs,), -1, dtype=torch.int64, device="cuda")
    infs = torch.full((m,), 255, dtype=torch.uint8, device="cuda")
    with eccmi.Context(0) as ctx:
        eccmi.ecc_msm_batch(ctx, c.cid, dev(bases), dev(s), offs, outs, infs,
                            flags=0 if endo else eccmi.ECC_NO_ENDOMORPHISM, window_c=wc)
        torch.cuda.synchronize()
    got = rows_to_points(c, outs.cpu().numpy().view(np.uint64).reshape(m, -1), infs.cpu().numpy())
    assert got == rows_to_points(c, out, inf)


@pytest.mark.parametrize("name", ["bn254", "bls12_381"])
@pytest.mark.parametrize("endo", [True, False])
@pytest.mark.parametrize("wc", [12, 13, 14, 15, 16, 17])
def test_reduction_lanes(name, wc, endo):
    """Buckets per reduction chain and lanes per addition across the widths at
    which the host's choice of them changes, alone and as part of a batch."""
    c = curves.CURVES[name]
    n = 300
    _, bases = seeded_bases(name, n, 941)
    s = seeded_scalars(name, n, 942, kind="bits")
    s[0] = syn.ints_to_limbs([(1 << c.scalar_bits) - 1], 4)[0]
    flags = 0 if endo else eccmi.ECC_NO_ENDOMORPHISM
    bd, sd = dev(bases), dev(s)
    out, inf = torch.zeros(2 * c.limbs, dtype=torch.int64, device="cuda"), torch.zeros(1, dtype=torch.uint8, device="cuda")
    offs = np.array([0, 100, 101, n], dtype=np.uint64)
    outs, infs = torch.zeros(6 * c.limbs, dtype=torch.int64, device="cuda"), torch.zeros(3, dtype=torch.uint8, device="cuda")
    with eccmi.Context(0) as ctx:
        eccmi.ecc_msm(ctx, c.cid, bd, sd, n, out, inf, flags=flags, window_c=wc)
        eccmi.ecc_msm_batch(ctx, c.cid, bd, sd, offs, outs, infs, flags=flags, window_c=wc)
        torch.cuda.synchronize()
    want, winf = co.msm_batch(c.cid, c.limbs, bases, s, np.array([0, n], dtype=np.uint64))
    bwant, bwinf = co.msm_batch(c.cid, c.limbs, bases, s, offs)
    assert rows_to_points(c, out.cpu().numpy().view(np.uint64).reshape(1, -1), inf.cpu().numpy()) == \
        rows_to_points(c, want, winf)
    assert rows_to_points(c, outs.cpu().numpy().view(np.uint64).reshape(3, -1), infs.cpu().numpy()) == \
        rows_to_points(c, bwant, bwinf)

"""Edges of the signed 4-bit windows of the per-lane point multiplication:
digits -8, -1, 0 and 7 at the bottom, in the middle and at the top, the carry
into digit 64, and sums that meet +-(a table entry) or O on the way, against
the CPU oracle, exactly."""

import numpy as np
import pytest

import synthetic as syn
from oracle import c_oracle as co
from oracle import curves
from tests.common import seeded_bases

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
eccmi = pytest.importorskip("paper_2501_03245_amd")


def window_edges(c):
    r, top = c.r, (1 << 256) - 1
    rep = [int(str(d) * 64, 16) for d in (7, 8)] + [int("78" * 32, 16), int("87" * 32, 16), int("f0" * 32, 16)]
    one = [d << s for d in (7, 8, 9, 15, 16, 17) for s in (0, 4, 124, 128, 248, 252)]
    # k P = (d 16^j) P + (r - d 16^j) P: the running sum passes through or next to O
    wrap = [(r + e) * m for e in (-9, -8, -7, -1, 0, 1, 7, 8, 9) for m in (1, 2, 15)]
    # around every multiple of the order below 2^256
    multi = [m * r + e for m in range(1, top // r + 1) for e in (-1, 0, 1)]
    return [v & top for v in rep + one + wrap + multi + [top, top - 7, top - 8, 1 << 255, (1 << 255) - 1, 0, 8 * r + 8]]


@pytest.mark.parametrize("name", ["bn254", "bls12_381", "secp256r1", "sm2"])
@pytest.mark.parametrize("pad", [0, 1, 63])
def test_signed_window_edges(name, pad):
    c = curves.CURVES[name]
    ks = syn.ints_to_limbs(window_edges(c) + [3] * pad, 4)
    n = ks.shape[0]
    _, pts = seeded_bases(name, n, 77 + pad)
    out, inf = co.scalar_mul(c.cid, c.limbs, ks, pts)
    want = out.copy()
    want[inf.astype(bool)] = 0
    got = torch.full((n * 2 * c.limbs,), -1, dtype=torch.int64, device="cuda")
    with eccmi.Context(0) as ctx:
        eccmi.ecc_pmul_batch(ctx, c.cid, torch.from_numpy(np.ascontiguousarray(pts).view(np.int64)).cuda(),
                             torch.from_numpy(ks.view(np.int64)).cuda(), n, got)
        torch.cuda.synchronize()
    assert np.array_equal(got.cpu().numpy().view(np.uint64).reshape(n, -1), want)

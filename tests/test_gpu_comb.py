"""Edges of the signed comb digits of the fixed-point multiplication (13-bit
windows; 8-bit ones in a context with an HBM budget): the most negative, zero
and most positive digit of single windows and of all, and the carry beyond bit
255, against the CPU oracle, exactly."""

import numpy as np
import pytest

import synthetic as syn
from oracle import c_oracle as co
from oracle import curves

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
eccmi = pytest.importorskip("paper_2501_03245_amd")


def digit_edges(c, w):
    top = (1 << 256) - 1
    half = 1 << (w - 1)
    one = [(half + e) << (w * j) for j in (0, 1, 7, 255 // w - 1, 255 // w) for e in (-2, -1, 0, 1)]
    every = [sum((half + e) << (w * j) for j in range(257 // w + 1)) for e in (-1, 0, 1)]
    return [v & top for v in one + every + [0, 1, 2, c.r - 1, c.r, c.r + 1, top, top - 1, 1 << 255, half, half - 1]]


@pytest.mark.parametrize("name", ["bn254", "bls12_381", "secp256r1", "sm2"])
@pytest.mark.parametrize("budget", [0, 1 << 28])
def test_comb_digit_edges(name, budget):
    c = curves.CURVES[name]
    ks = syn.ints_to_limbs(digit_edges(c, 13) + digit_edges(c, 8), 4)
    n = ks.shape[0]
    want = co.fixed_base(c.cid, c.limbs, ks)
    got = torch.full((n * 2 * c.limbs,), -1, dtype=torch.int64, device="cuda")
    with eccmi.Context(0, hbm_budget_bytes=budget) as ctx:
        eccmi.ecc_fixed_base_mul(ctx, c.cid, torch.from_numpy(ks.view(np.int64)).cuda(), n, got)
        torch.cuda.synchronize()
    assert np.array_equal(got.cpu().numpy().view(np.uint64).reshape(n, -1), want)

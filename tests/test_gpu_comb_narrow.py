"""Edges of the 9-bit comb digits of a context with an HBM budget, on one lane
per request and on four, against the CPU oracle, exactly."""

import numpy as np
import pytest

import synthetic as syn
from oracle import c_oracle as co
from oracle import curves
from tests.test_gpu_comb import digit_edges

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
eccmi = pytest.importorskip("paper_2501_03245_amd")


@pytest.mark.parametrize("name", ["bn254", "bls12_381", "secp256r1", "sm2"])
@pytest.mark.parametrize("n", [1, 16384, 16385])
def test_narrow_digit_edges(name, n):
    c = curves.CURVES[name]
    edges = digit_edges(c, 9)
    want = co.fixed_base(c.cid, c.limbs, syn.ints_to_limbs(edges, 4))
    i = np.arange(n) % len(edges)
    ks = syn.ints_to_limbs(edges, 4)[i]
    got = torch.full((n * 2 * c.limbs,), -1, dtype=torch.int64, device="cuda")
    with eccmi.Context(0, hbm_budget_bytes=1 << 28) as ctx:
        eccmi.ecc_fixed_base_mul(ctx, c.cid, torch.from_numpy(ks.view(np.int64)).cuda(), n, got)
        torch.cuda.synchronize()
    assert np.array_equal(got.cpu().numpy().view(np.uint64).reshape(n, -1), want[i])

"""Both sides of the size at which a request moves from four lanes to one: a
call of n requests against the same requests in two calls of at most 2^14, and
a sample of them against the CPU oracle, exactly.  Scalars hold the digits'
edges."""

import numpy as np
import pytest

import synthetic as syn
from oracle import c_oracle as co
from oracle import curves
from tests.common import seeded_signatures
from tests.test_gpu_comb import digit_edges
from tests.test_gpu_signed_windows import window_edges

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
eccmi = pytest.importorskip("paper_2501_03245_amd")

EDGE = 1 << 14


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a).view(np.int64)).cuda()


def in_two(n, call):
    """call(lo, hi) for the whole range and for two halves; both results."""
    h = n // 2
    return call(0, n), torch.cat([call(0, h), call(h, n)])


@pytest.mark.parametrize("name", ["bn254", "bls12_381", "secp256r1", "sm2"])
@pytest.mark.parametrize("n", [EDGE, EDGE + 1, EDGE + 64])
def test_products_across_the_edge(name, n):
    c = curves.CURVES[name]
    edges = syn.ints_to_limbs(window_edges(c) + digit_edges(c, 13), 4)
    ks = syn.uniform_bits(0x9AD, syn.TAG_SCALARS, n, 256, 4)
    ks[: len(edges)] = edges
    ks[n - len(edges):] = edges
    td = dev(syn.uniform_range(0x9AE, syn.TAG_BASE_DLOG, n, 1, c.r, 4))
    tk = dev(ks)
    with eccmi.Context(0) as ctx:
        def fixed(s, lo, hi):
            out = torch.zeros((hi - lo, 2 * c.limbs), dtype=torch.int64, device="cuda")
            eccmi.ecc_fixed_base_mul(ctx, c.cid, s[lo:hi].contiguous(), hi - lo, out)
            return out

        pts, pts2 = in_two(n, lambda lo, hi: fixed(td, lo, hi))
        assert torch.equal(pts, pts2)
        g, g2 = in_two(n, lambda lo, hi: fixed(tk, lo, hi))
        assert torch.equal(g, g2)

        def pmul(lo, hi):
            out = torch.zeros((hi - lo, 2 * c.limbs), dtype=torch.int64, device="cuda")
            eccmi.ecc_pmul_batch(ctx, c.cid, pts[lo:hi].contiguous(), tk[lo:hi].contiguous(), hi - lo, out)
            return out

        a, b = in_two(n, pmul)
        assert torch.equal(a, b)
    at = np.r_[0:len(edges), n - 8:n]
    want, inf = co.scalar_mul(c.cid, c.limbs, ks[at], pts.cpu().numpy().view(np.uint64)[at])
    want = want.copy()
    want[inf.astype(bool)] = 0
    assert np.array_equal(a.cpu().numpy().view(np.uint64)[at], want)


@pytest.mark.parametrize("name", ["secp256r1", "sm2"])
@pytest.mark.parametrize("n", [EDGE, EDGE + 1])
def test_signatures_across_the_edge(name, n):
    c = curves.CURVES[name]
    d = syn.uniform_range(0x51, syn.TAG_KEYS, n, 1, c.r, 4)
    k = syn.uniform_range(0x52, syn.TAG_NONCES, n, 1, c.r, 4)
    d[3] = 0  # out of range: r = s = 0, and no signature verifies
    k[n - 2] = syn.ints_to_limbs([c.r], 4)[0]
    h = torch.from_numpy(syn.random_bytes(0x53, syn.TAG_HASH, n, 32)).cuda()
    td, tk = dev(d), dev(k)
    with eccmi.Context(0) as ctx:
        def sign(lo, hi):
            out = torch.zeros((hi - lo, 8), dtype=torch.int64, device="cuda")
            eccmi.ecc_sign_batch(ctx, c.cid, h[lo:hi].contiguous(), td[lo:hi].contiguous(), tk[lo:hi].contiguous(),
                                 hi - lo, out)
            return out

        sigs, sigs2 = in_two(n, sign)
        assert torch.equal(sigs, sigs2)
        pub = torch.zeros((n, 8), dtype=torch.int64, device="cuda")
        eccmi.ecc_fixed_base_mul(ctx, c.cid, td, n, pub)
        forged = h.clone()
        forged[::16, 5] ^= 1

        def verify(lo, hi):
            out = torch.full((hi - lo,), 7, dtype=torch.uint8, device="cuda")
            eccmi.ecc_verify_batch(ctx, c.cid, forged[lo:hi].contiguous(), pub[lo:hi].contiguous(),
                                   sigs[lo:hi].contiguous(), hi - lo, out)
            return out

        v, v2 = in_two(n, verify)
    assert torch.equal(v, v2)
    want = np.ones(n, dtype=np.uint8)
    want[::16] = 0
    want[[3, n - 2]] = 0
    assert np.array_equal(v.cpu().numpy(), want)


@pytest.mark.parametrize("m", [1, 15, 16, 17, 64, 65])
def test_small_verifications(m):
    hashes, pub, sigs = seeded_signatures(m, 0x71 + m, corrupt_every=3)
    want = co.ecdsa_verify(eccmi.ECC_SECP256R1, hashes, pub, sigs)
    with eccmi.Context(0) as ctx:
        got = {}
        for form in (eccmi.ECC_VERIFY_PER_LANE, eccmi.ECC_VERIFY_BATCHED):
            out = torch.full((m,), 7, dtype=torch.uint8, device="cuda")
            eccmi.ecc_verify_batch(ctx, eccmi.ECC_SECP256R1, torch.from_numpy(hashes).cuda(), dev(pub), dev(sigs), m,
                                   out, flags=form)
            got[form] = out.cpu().numpy()
    assert np.array_equal(got[eccmi.ECC_VERIFY_PER_LANE], got[eccmi.ECC_VERIFY_BATCHED])
    assert np.array_equal(got[eccmi.ECC_VERIFY_PER_LANE], want)

"""The calls whose speed this library is judged by, each through a public entry point.

A case names an entry point (`kind`), a curve, a size and the call's options:

    msm     one multi-scalar multiplication of `n` points (a commitment in a proof system)
    batch   `n` independent MSMs of 2**lo .. 2**hi points each, sizes log-uniform, in one call
    verify  `n` ECDSA verifications, about every 16th request forged
    sign    `n` ECDSA signatures
    pmul    `n` products k_i P_i of run-time points (key agreement)
    fpmul   `n` products k_i G of the generator (key generation)

Inputs are resident on the GPU, or in host memory where `host` is true.  The
context, with the tables it makes on its first call, is kept for the life of
the process, as a service keeps it.
"""

from __future__ import annotations

import math

import numpy as np
import torch

import paper_2501_03245_amd as eccmi

CURVE_ID = eccmi.CURVES

# prime, group order, a, generator (published parameters)
PARAMS = {
    "bn254": (0x30644E72E131A029B85045B68181585D97816A916871CA8D3C208C16D87CFD47,
              0x30644E72E131A029B85045B68181585D2833E84879B9709143E1F593F0000001, 0, 1, 2),
    "bls12_381": (0x1A0111EA397FE69A4B1BA7B6434BACD764774B84F38512BF6730D2A0F6B0F6241EABFFFEB153FFFFB9FEFFFFFFFFAAAB,
                  0x73EDA753299D7D483339D80809A1D80553BDA402FFFE5BFEFFFFFFFF00000001, 0,
                  0x17F1D3A73197D7942695638C4FA9AC0FC3688C4F9774B905A14E3A3F171BAC586C55E83FF97A1AEFFB3AF00ADB22C6BB,
                  0x08B3F481E3AAA0F1A09E30ED741D8AE4FCF5E095D5D00AF600DB18CB2C04B3EDD03CC744A2888AE40CAA232946C5E7E1),
    "secp256r1": (0xFFFFFFFF00000001000000000000000000000000FFFFFFFFFFFFFFFFFFFFFFFF,
                  0xFFFFFFFF00000000FFFFFFFFFFFFFFFFBCE6FAADA7179E84F3B9CAC2FC632551, -3,
                  0x6B17D1F2E12C4247F8BCE6E563A440F277037D812DEB33A0F4A13945D898C296,
                  0x4FE342E2FE1A7F9B8EE7EB4A7C0F9E162BCE33576B315ECECBB6406837BF51F5),
    "sm2": (0xFFFFFFFEFFFFFFFFFFFFFFFFFFFFFFFFFFFFFFFF00000000FFFFFFFFFFFFFFFF,
            0xFFFFFFFEFFFFFFFFFFFFFFFFFFFFFFFF7203DF6B21C6052B53BBF40939D54123, -3,
            0x32C4AE2C1F1981195F9904466A39C9948FE30BBFF2660BE1715A4589334C74C7,
            0xBC3736A2F4F6779C59BDCEE36B692153D0A9877CC62A474002DF32E52139F0A0),
}

# multiply-adds of 32-bit words in one Montgomery product of m words: 2 m^2 + m
MADS = {"bn254": 136, "bls12_381": 300, "secp256r1": 136, "sm2": 136}


def _case(name, kind, curve, n, **more):
    c = {"name": name, "kind": kind, "curve": curve, "n": n, "mont": False, "check": False, "host": False, "lo": 0,
         "hi": 0}
    c.update(more)
    return c


def listed():
    return [
        # a small circuit's commitment, its bases kept in Montgomery form: all fixed costs
        _case("msm-bn254-4k", "msm", "bn254", 4096, mont=True),
        # the smallest requests of the served mix, at a ragged size
        _case("msm-bls-1k", "msm", "bls12_381", 1021),
        # a medium commitment, where fixed costs and throughput weigh alike
        _case("msm-bls-64k", "msm", "bls12_381", 1 << 16),
        # the headline size: one large commitment
        _case("msm-bls-1m", "msm", "bls12_381", 1 << 20),
        # a large commitment of no round size over bases that are not trusted
        _case("msm-bn254-700k", "msm", "bn254", 700001, check=True),
        # many provers' commitments of uneven sizes in one call
        _case("batch-bls-512", "batch", "bls12_381", 512, lo=1, hi=14),
        # one batch of a verification service at low load: latency
        _case("verify-p256-256", "verify", "secp256r1", 256),
        # a block's worth of signatures: throughput
        _case("verify-sm2-64k", "verify", "sm2", 1 << 16),
        # bulk signing
        _case("sign-sm2-256k", "sign", "sm2", 1 << 18),
        # bulk key agreement, the smallest batch of the paper's throughput table
        _case("pmul-sm2-512k", "pmul", "sm2", 1 << 19),
        # key agreement or re-randomisation over a few thousand points on a pairing curve
        _case("pmul-bn254-3k", "pmul", "bn254", 3001),
        # bulk key generation, the smallest batch of the paper's throughput table
        _case("fpmul-sm2-512k", "fpmul", "sm2", 1 << 19),
    ]


def _log_size(rng, lo, hi):
    n = int(round(2.0 ** rng.uniform(math.log2(lo), math.log2(hi))))
    return max(lo, min(hi, n))


def draw(rng):
    """One more case: any curve a call takes, sizes log-uniform from tens of requests to the listed largest."""
    kind = rng.choice(["msm", "msm", "msm", "batch", "verify", "verify", "sign", "pmul", "pmul", "fpmul"])
    if kind in ("msm", "batch"):
        curve = rng.choice(["bn254", "bls12_381"])
    elif kind in ("verify", "sign"):
        curve = rng.choice(["secp256r1", "sm2"])
    else:
        curve = rng.choice(["bn254", "bls12_381", "secp256r1", "sm2"])
    c = _case("", kind, curve, 0)
    del c["name"]
    c["host"] = rng.random() < 0.2
    if kind == "msm":
        c["n"] = _log_size(rng, 64, 1 << 20)
        c["mont"] = rng.random() < 0.3
        c["check"] = rng.random() < 0.3
    elif kind == "batch":
        c["lo"] = rng.randrange(1, 5)
        c["hi"] = rng.randrange(8, 15)
        c["n"] = _log_size(rng, 4, 512)
    elif kind == "pmul":
        c["n"] = _log_size(rng, 32, {"bls12_381": 1 << 17, "bn254": 1 << 18}.get(curve, 1 << 19))
    elif kind == "fpmul":
        c["n"] = _log_size(rng, 32, 1 << 18 if curve == "bls12_381" else 1 << 19)
    else:
        c["n"] = _log_size(rng, 32, 1 << 18)
    return c


# ---- inputs ---------------------------------------------------------------------


def _words(seed, stream, n, k):
    """n rows of k random 64-bit words on the GPU, from the seed and a stream number alone."""
    g = torch.Generator(device="cuda")
    g.manual_seed(seed * 64 + stream)
    return torch.randint(-(1 << 63), (1 << 63) - 1, (n, k), dtype=torch.int64, device="cuda", generator=g)


def _below(seed, stream, n, bound):
    """n integers of four words, uniform below the bound up to the bound's lowest 192 bits."""
    w = _words(seed, stream, n, 4)
    top = bound >> 192
    w[:, 3] = torch.remainder((w[:, 3] >> 1) & ((1 << 63) - 1), min(top, (1 << 63) - 1))
    return w


def _scalars(case, seed, n):
    """MSM scalars: uniform 255-bit integers on BLS12-381, uniform below the group order on BN254."""
    if case["curve"] == "bls12_381":
        w = _words(seed, 1, n, 4)
        w[:, 3] &= (1 << 63) - 1
        return w
    return _below(seed, 1, n, PARAMS["bn254"][1])


def _batch_offsets(case, seed):
    rng = np.random.default_rng(seed)
    sizes = np.rint(np.exp2(rng.uniform(case["lo"], case["hi"], case["n"]))).astype(np.int64)
    return np.concatenate([[0], np.cumsum(sizes)]).astype(np.uint64)


def _total(case, seed):
    return int(_batch_offsets(case, seed)[-1]) if case["kind"] == "batch" else case["n"]


_CTX = {}


def _ctx():
    if 0 not in _CTX:
        _CTX[0] = eccmi.Context(0)
    return _CTX[0]


def _points(curve, ks, mont=False):
    cid = CURVE_ID[curve]
    out = torch.empty((ks.shape[0], 2 * eccmi.LIMBS[cid]), dtype=torch.int64, device="cuda")
    eccmi.ecc_fixed_base_mul(_ctx(), cid, ks, ks.shape[0], out, flags=eccmi.ECC_IN_MONTGOMERY if mont else 0)
    return out


def _empty(rows, words, dtype=torch.int64):
    return torch.zeros((rows, words) if words else (rows,), dtype=dtype, device="cuda")


def _forged(seed, n):
    return (_words(seed, 5, n, 1)[:, 0] & 15) == 0


def prepare(case, seed):
    kind, curve, n = case["kind"], case["curve"], case["n"]
    cid = CURVE_ID[curve]
    words = 2 * eccmi.LIMBS[cid]
    order = PARAMS[curve][1]
    s = {"case": case, "cid": cid, "n": n}
    if kind in ("msm", "batch"):
        total = _total(case, seed)
        s["points"] = _points(curve, _below(seed, 2, total, order), case["mont"])
        s["scalars"] = _scalars(case, seed, total)
        m = n if kind == "batch" else 1
        s["out"], s["inf"] = _empty(m, words), _empty(m, 0, torch.uint8)
        if kind == "batch":
            s["offsets"] = _batch_offsets(case, seed)
        s["flags"] = (eccmi.ECC_IN_MONTGOMERY if case["mont"] else 0) | (eccmi.ECC_CHECK_ON_CURVE if case["check"] else 0)
    elif kind in ("verify", "sign"):
        keys, nonces = _below(seed, 2, n, order), _below(seed, 3, n, order)
        hashes = _words(seed, 4, n, 4).view(torch.uint8)
        s["sigs"] = _empty(n, 8)
        if kind == "sign":
            s["hashes"], s["keys"], s["nonces"] = hashes, keys, nonces
        else:
            eccmi.ecc_sign_batch(_ctx(), cid, hashes, keys, nonces, n, s["sigs"])
            s["points"] = _points(curve, keys)
            hashes[_forged(seed, n), 7] ^= 1
            s["hashes"], s["valid"] = hashes, _empty(n, 0, torch.uint8)
    elif kind == "pmul":
        s["points"], s["scalars"], s["out"] = _points(curve, _below(seed, 2, n, order)), _words(seed, 1, n, 4), _empty(n, words)
    else:
        s["scalars"], s["out"] = _words(seed, 1, n, 4), _empty(n, words)
    if case["host"]:
        s = {k: v.cpu().numpy() if isinstance(v, torch.Tensor) else v for k, v in s.items()}
    return s


def run(s):
    kind, cid, n = s["case"]["kind"], s["cid"], s["n"]
    ctx = _ctx()
    if kind == "msm":
        eccmi.ecc_msm(ctx, cid, s["points"], s["scalars"], n, s["out"], s["inf"], flags=s["flags"])
        return {"out": s["out"], "inf": s["inf"]}
    if kind == "batch":
        eccmi.ecc_msm_batch(ctx, cid, s["points"], s["scalars"], s["offsets"], s["out"], s["inf"], flags=s["flags"])
        return {"out": s["out"], "inf": s["inf"]}
    if kind == "verify":
        eccmi.ecc_verify_batch(ctx, cid, s["hashes"], s["points"], s["sigs"], n, s["valid"])
        return {"valid": s["valid"]}
    if kind == "sign":
        eccmi.ecc_sign_batch(ctx, cid, s["hashes"], s["keys"], s["nonces"], n, s["sigs"])
        return {"sigs": s["sigs"]}
    if kind == "pmul":
        eccmi.ecc_pmul_batch(ctx, cid, s["points"], s["scalars"], n, s["out"])
    else:
        eccmi.ecc_fixed_base_mul(ctx, cid, s["scalars"], n, s["out"])
    return {"out": s["out"]}


# ---- what a pass cannot do without -------------------------------------------------


def _msm_products(n):
    """Field products of n points' windowed sum: half-length scalars of the endomorphism, the best window width,
    six products for an affine addition that shares its inversion and twelve per bucket for the running sums."""
    return min(math.ceil(128 / c) * (2 * n * 6 + (1 << (c - 1)) * 2 * 12) for c in range(2, 20))


def work(case):
    kind, n, curve = case["kind"], case["n"], case["curve"]
    pt = 16 * eccmi.LIMBS[CURVE_ID[curve]]
    comb = 20 * 10  # k G: 20 mixed additions from a table of the generator's multiples
    # k P: 256 doublings of 8 products and 52 additions of 11; half the doublings where an endomorphism holds everywhere
    free = (128 if curve == "bn254" else 256) * 8 + 52 * 11
    if kind == "msm":
        products, nbytes = _msm_products(n), n * (pt + 32) + pt + 1
    elif kind == "batch":
        # sizes are log-uniform: the mean over eight equal steps of the exponent
        sizes = [2.0 ** (case["lo"] + (case["hi"] - case["lo"]) * (i + 0.5) / 8) for i in range(8)]
        products = n * sum(_msm_products(x) for x in sizes) / 8
        nbytes = n * (sum(sizes) / 8 * (pt + 32) + pt + 1)
    elif kind == "verify":
        products, nbytes = n * (free + comb), n * (32 + 64 + 64 + 1)
    elif kind == "sign":
        products, nbytes = n * comb, n * (32 + 32 + 32 + 64)
    elif kind == "pmul":
        products, nbytes = n * free, n * (2 * pt + 32)
    else:
        products, nbytes = n * comb, n * (pt + 32)
    return {"bytes": float(nbytes), "flops": 2.0 * MADS[curve] * products}


# ---- the same results in plain integers --------------------------------------------


def _ints(rows):
    rows = np.ascontiguousarray(rows.cpu().numpy()).view(np.uint64)
    k = rows.shape[1] * 8
    raw = rows.astype("<u8").tobytes()
    return [int.from_bytes(raw[i:i + k], "little") for i in range(0, len(raw), k)]


def _mul_g(curve, k):
    """k G by double-and-add in Jacobian coordinates; None for the point at infinity."""
    p, r, a, gx, gy = PARAMS[curve]
    k %= r
    X, Y, Z = 0, 1, 0
    for bit in bin(k)[2:] if k else "":
        if Z:
            yy = Y * Y % p
            s4 = 4 * X * yy % p
            m = (3 * X * X + a * pow(Z, 4, p)) % p
            Z = 2 * Y * Z % p
            X = (m * m - 2 * s4) % p
            Y = (m * (s4 - X) - 8 * yy * yy) % p
        if bit == "1":
            if not Z:
                X, Y, Z = gx, gy, 1
                continue
            zz = Z * Z % p
            h, t = (gx * zz - X) % p, (gy * zz * Z - Y) % p
            if h == 0:  # the same point: 2 G, reached only at k = 2 after an addition of G to itself
                raise ArithmeticError("addition of equal points")
            hh = h * h % p
            v, hhh = X * hh % p, h * hh % p
            X = (t * t - hhh - 2 * v) % p
            Y = (t * (v - X) - Y * hhh) % p
            Z = Z * h % p
    if not Z:
        return None
    zi = pow(Z, -1, p)
    return X * zi * zi % p, Y * zi * zi * zi % p


def _limb_rows(values, k, host):
    raw = b"".join(v.to_bytes(8 * k, "little") for v in values)
    a = np.frombuffer(raw, dtype=np.int64).reshape(len(values), k).copy()
    return a if host else torch.from_numpy(a).cuda()


def _point_rows(points, limbs, host):
    return _limb_rows([0 if q is None else q[0] | (q[1] << (64 * limbs)) for q in points], 2 * limbs, host)


def exact(case, seed):
    kind, curve, n, host = case["kind"], case["curve"], case["n"], case["host"]
    limbs = eccmi.LIMBS[CURVE_ID[curve]]
    order = PARAMS[curve][1]

    def flags(values):
        a = np.array(values, dtype=np.uint8)
        return a if host else torch.from_numpy(a).cuda()

    if kind in ("msm", "batch"):
        total = _total(case, seed)
        ks, ss = _ints(_below(seed, 2, total, order)), _ints(_scalars(case, seed, total))
        offs = [int(x) for x in _batch_offsets(case, seed)] if kind == "batch" else [0, n]
        pts = [_mul_g(curve, sum(k * s for k, s in zip(ks[a:b], ss[a:b]))) for a, b in zip(offs, offs[1:])]
        return {"out": _point_rows(pts, limbs, host), "inf": flags([q is None for q in pts])}
    if kind == "verify":
        return {"valid": flags((~_forged(seed, n)).cpu().numpy())}
    if n > 4096:
        return None
    if kind == "sign":
        ds, ns = _ints(_below(seed, 2, n, order)), _ints(_below(seed, 3, n, order))
        es = [int.from_bytes(bytes(h), "big") for h in _words(seed, 4, n, 4).view(torch.uint8).cpu().numpy()]
        rows = []
        for d, k, e in zip(ds, ns, es):
            r = _mul_g(curve, k)[0] % order
            rows.append(r | (pow(k, -1, order) * (e + r * d) % order) << 256)
        return {"sigs": _limb_rows(rows, 8, host)}
    ks = _ints(_words(seed, 1, n, 4))
    if kind == "pmul":
        ks = [k * b for k, b in zip(ks, _ints(_below(seed, 2, n, order)))]
    return {"out": _point_rows([_mul_g(curve, k) for k in ks], limbs, host)}

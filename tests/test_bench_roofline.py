"""The bench's roofline entry: priced by the form of the bucket accumulation that
ran, its traffic figure tied to every header the kernels are built from."""

import os
import re

import bench

CSRC = os.path.join(bench.ROOT, "paper_2501_03245_amd", "csrc")


def stats(launches):
    return {"msm_calls": 2, "points": 2 << 20, "round_launches": launches, "round_adds": 3 * 10**7, "round_ms": 5.0,
            "finish_ms": 0.5}


def test_direct_sums_and_rounds_are_priced_apart():
    direct = bench.accumulation_roofline(stats(2), 2, 2, 1 << 24)
    rounds = bench.accumulation_roofline(stats(40), 2, 2, 1 << 24)
    assert direct["kernel"].startswith("k_bucket_acc ") and rounds["kernel"].startswith("k_bucket_round ")
    assert direct["achieved"] * bench.MULS_PER_AFFINE_ADD == rounds["achieved"] * bench.MULS_PER_XYZZ_ADD
    assert direct["traffic"] is None and rounds["traffic"] is None  # counted at 2^20 points only


def test_traffic_follows_every_source():
    seen, todo = set(), ["accumulate.h"]
    while todo:
        name = todo.pop()
        if name in seen:
            continue
        seen.add(name)
        with open(os.path.join(CSRC, name)) as f:
            todo += re.findall(r'#include "(\w+\.h)"', f.read())
    assert seen == set(bench.KERNEL_SOURCES)

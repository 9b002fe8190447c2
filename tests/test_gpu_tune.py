"""The tuner: the rounds' parameters are measured only where the rounds run, and
what it finds for one MSM alone leaves the MSMs of a batch their own width."""

import numpy as np
import pytest

from oracle import curves

pytestmark = pytest.mark.gpu

pytest.importorskip("torch")
eccmi = pytest.importorskip("paper_2501_03245_amd")


@pytest.mark.parametrize("name", ["bn254", "bls12_381"])
def test_rounds_parameters_stay_where_no_round_runs(name):
    cid = curves.CURVES[name].cid
    with eccmi.Context(0) as ctx:
        before = [eccmi.ecc_tuned_params(ctx, cid, 1 << lg)[1] for lg in range(5, 13)]
        eccmi.ecc_tune(ctx, cid, 5, 12, reps=3)
        assert [eccmi.ecc_tuned_params(ctx, cid, 1 << lg)[1] for lg in range(5, 13)] == before


@pytest.mark.parametrize("name", ["bn254", "bls12_381"])
def test_batches_keep_their_width(name, tmp_path):
    cid = curves.CURVES[name].cid
    offs = np.arange(65, dtype=np.uint64) * 100
    path = str(tmp_path / "tune.txt")
    with eccmi.Context(0) as ctx:
        own = eccmi.ecc_msm_batch_scratch_bytes(ctx, cid, offs)
        one = eccmi.ecc_msm_batch_scratch_bytes(ctx, cid, offs[:2])
        eccmi.ecc_tune(ctx, cid, 6, 6, reps=1)
        eccmi.ecc_tune_save(ctx, path)
        with open(path) as f:
            lines = [line.split() for line in f if not line.startswith("#")]
        with open(path, "w") as f:
            f.writelines(" ".join(x[:3] + ["13"] + x[4:]) + "\n" for x in lines)
        assert eccmi.ecc_tune_load(ctx, path) == 1
        assert eccmi.ecc_tuned_params(ctx, cid, 100)[0] == 13
        assert eccmi.ecc_msm_batch_scratch_bytes(ctx, cid, offs) == own
        assert eccmi.ecc_msm_batch_scratch_bytes(ctx, cid, offs[:2]) != one  # one MSM follows the table

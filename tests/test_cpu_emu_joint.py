"""Joint frames of a batch that are narrower than a workgroup (several rows of
the upsampling go side by side), on the host: against the oracle, and the
persistent launch against one launch per stage, bit for bit."""
import pytest

from tests.cpu_emu.harness import run_in_subprocess


@pytest.mark.parametrize("joint,up", [([52, 2], 2), ([19 * 4, 64], 4), ([22, 130], 2),
                                      ([36, 128], 2)])
def test_emulated_narrow_joint(joint, up):
    res = run_in_subprocess(dict(kind="batch", H=0, W=0, Q=8, C=3, r=4, sizes=[[5, 20]],
                                 joint=joint, up=up))
    assert res["persistent_not_failed"] and res["persistent_equals_stages"], res
    assert res["plain0_equal"] and res["joint_rel"] <= 1e-6, res

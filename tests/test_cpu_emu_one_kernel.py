"""The fused path's one-kernel form on the host: frames and segments whose ring
is smaller than the coefficient image, so that the least workspace selects it.
Against the oracle at the FP32 path's tolerance, and two of them under
AddressSanitizer and UndefinedBehaviorSanitizer."""
import pytest

from tests.cpu_emu.harness import run_in_subprocess

CASES = [
    # two strips and two segments of the RGB workload
    dict(kind="one_kernel", H=60, W=300, Q=8, C=3, r=8, tile_rows=30, frame="config", config=1),
    # wide prefix segments, the Appendix's regulariser
    dict(kind="one_kernel", H=110, W=210, Q=4, C=1, r=16, tile_rows=110, mode="paper",
         eps_mul=0.2, offset=2.0),
    # vertical sums outside LDS
    dict(kind="one_kernel", H=30, W=120, Q=8, C=4, r=3, tile_rows=15),
]
SANITIZED = [
    dict(kind="one_kernel", H=24, W=255, Q=3, C=1, r=2, tile_rows=12),
    dict(kind="one_kernel", H=40, W=200, Q=2, C=1, r=9, tile_rows=40, mode="paper", eps_mul=0.1),
]


def _check(res):
    assert res["one_kernel"] is True and res["fused_rel"] <= 1e-4, res


def _id(spec):
    return "-".join(f"{k}{spec[k]}" for k in ("H", "W", "Q", "C", "r"))


@pytest.mark.parametrize("spec", CASES, ids=_id)
def test_emulated_one_kernel(spec):
    _check(run_in_subprocess(spec))


@pytest.mark.parametrize("spec", SANITIZED, ids=_id)
def test_sanitized_one_kernel(spec):
    _check(run_in_subprocess(spec, sanitize=True, timeout=900))

"""flr_batch_plan on the host: the plan keeps the caller's parameters."""
from tests.cpu_emu.harness import run_in_subprocess


def test_plan_params_are_the_callers():
    res = run_in_subprocess(dict(kind="batch_plan", H=0, W=0, Q=3, C=1, r=2,
                                 sizes=[[9, 30], [40, 70]], tile_rows=5))
    assert res["tile_rows"] == 5 and res["plan_tile_rows"] == 5, res
    assert res["avg_rows"] == 2, res

"""What a changed source invalidates: the emulator's build and the bench's
counter figures."""
import os
import re

from tests.cpu_emu import harness


def _includes(path, dirs):
    out, todo = set(), [path]
    while todo:
        for name in re.findall(r'^\s*#include\s+"([^"]+)"', open(todo.pop()).read(), re.M):
            for d in dirs:
                p = os.path.join(d, name)
                if os.path.exists(p) and p not in out:
                    out.add(p)
                    todo.append(p)
    return out


def test_emulator_is_rebuilt_for_every_file_it_compiles():
    deps = {os.path.realpath(p) for p in harness.dependencies()}
    need = set(harness.UNITS)
    for u in harness.UNITS:
        need |= _includes(u, (harness.CSRC, harness.INCLUDE, harness.HERE))
    assert {os.path.realpath(p) for p in need} <= deps


def test_counter_digest_covers_the_launched_kernels():
    """flr_q08.hip holds the walkers, flr_adjoint.hip the averaging."""
    import bench
    csrc = os.path.join(harness.ROOT, "paper_2410_11625_amd", "csrc")
    units = [f for f in bench.COUNTED_SOURCES if f.endswith(".hip")]
    assert "apply_avg_kernel" in open(os.path.join(csrc, "flr_adjoint.hip")).read()
    assert set(units) == {"flr_q08.hip", "flr_adjoint.hip"}
    for f in bench.COUNTED_SOURCES:
        assert os.path.exists(os.path.join(csrc, f))

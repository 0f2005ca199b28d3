"""What a changed source invalidates: the emulator's build."""
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


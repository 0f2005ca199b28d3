"""The registers that the built kernels hold, against what the launch planner
and the choice of kernel forms assume (read from libflr.so's kernel metadata
with the ROCm tools that built it; nothing runs)."""
import os
import re
import shutil
import subprocess

import pytest

from paper_2410_11625_amd import build as flr_build

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
LLVM = "/opt/rocm/llvm/bin"
MAGIC = b"__CLANG_OFFLOAD_BUNDLE__"


@pytest.fixture(scope="module")
def kernels(tmp_path_factory):
    """{demangled kernel: (registers, spilled registers)} of libflr.so."""
    objcopy, readelf = (os.path.join(LLVM, t) for t in ("llvm-objcopy", "llvm-readelf"))
    if not (os.path.exists(objcopy) and os.path.exists(readelf) and shutil.which("c++filt")):
        pytest.skip("no ROCm binary tools")
    tmp = tmp_path_factory.mktemp("co")
    fat = str(tmp / "fat")
    subprocess.run([objcopy, f"--dump-section=.hip_fatbin={fat}", flr_build.LIB,
                    str(tmp / "copy")], check=True)
    data = open(fat, "rb").read()
    found = {}
    at = data.find(MAGIC)
    while at >= 0:
        num = int.from_bytes(data[at + 24:at + 32], "little")
        pos = at + 32
        for _ in range(num):
            off, size, idlen = (int.from_bytes(data[pos + 8 * i:pos + 8 * i + 8], "little")
                                for i in range(3))
            name = data[pos + 24:pos + 24 + idlen].decode()
            pos += 24 + idlen
            if "gfx950" in name and size:
                co = str(tmp / "co")
                open(co, "wb").write(data[at + off:at + off + size])
                notes = subprocess.run([readelf, "--notes", co], check=True, capture_output=True,
                                       text=True).stdout
                for k in notes.split("- .agpr_count:")[1:]:
                    f = dict(re.findall(r"\.(\w+):\s+(\S+)", k))
                    found[f["name"]] = (int(f["vgpr_count"]), int(f["vgpr_spill_count"]))
        at = data.find(MAGIC, at + 1)
    assert found
    plain = subprocess.run(["c++filt"], input="\n".join(found), capture_output=True, text=True,
                           check=True).stdout.splitlines()
    return dict(zip(plain, found.values()))


def test_planned_workgroups_fit_the_registers(kernels, tmp_path):
    """Each workgroup of a walker has one wave on a SIMD's 512 registers
    (given out in eights): as many as the planner counts on fit."""
    src = tmp_path / "p.cpp"
    src.write_text("""#include "flr_launch.hpp"
#include <cstdio>
using namespace flr;
int main() {
  const int kinds[3] = {K_MOMENTS, K_FUSED0, K_COEFFS};
  for (int m = 0; m < 3; ++m)
    for (int Q = 1; Q <= 12; ++Q)
      for (int C = 1; C <= 4; ++C)
        std::printf("%d %d %d %d\\n", kinds[m] == K_COEFFS ? 3 : m, Q, C,
                    workgroups_per_cu(kinds[m], Q, C));
}
""")
    exe = str(tmp_path / "p")
    subprocess.run(["g++", "-std=c++20", "-w", "-I" + os.path.join(ROOT, "tests", "cpu_emu"),
                    "-I" + os.path.join(ROOT, "paper_2410_11625_amd", "csrc"), str(src), "-o",
                    exe], check=True)
    planned = {tuple(map(int, l.split()[:3])): int(l.split()[3]) for l in
               subprocess.run([exe], check=True, capture_output=True, text=True).stdout.splitlines()}
    checked = 0
    for name, (regs, _) in kernels.items():
        m = re.search(r"flr::walk_kernel<(\d+), (\d+), (\d+), \w+, 0, -1, \w+>", name)
        if m and int(m[3]) in (0, 1, 3):
            n = planned[int(m[3]), int(m[1]), int(m[2])]
            assert n * ((regs + 7) // 8 * 8) <= 512, (name, regs, n)
            checked += n > 1
    assert checked >= 50


def test_paired_walkers_hold_their_systems(kernels):
    """Where the solving waves spill much of a pixel's system, the unpaired
    walker is the faster one (measured: 56 registers are worth it, 129 not)."""
    pairs = {n: spill for n, (_, spill) in kernels.items() if "walk_pair_kernel<" in n}
    assert pairs and max(pairs.values()) <= 64, max(pairs, key=pairs.get)

"""Registers of the compiled decode kernels: the rules on sizes (csrc/mq_plan.h) count on two workgroups of eight waves, or sixteen waves in
all, sharing a compute unit, which takes 128 registers a wave at most."""
import os
import re
import shutil
import subprocess

import pytest

from paper_2502_06786_amd import build as mq_build
from tests import plans
from tests.test_matrix_waits import OBJDUMP

READELF = os.path.join(os.path.dirname(OBJDUMP), "llvm-readelf")


@pytest.fixture(scope="module")
def registers(tmp_path_factory):
    """kernel (mangled) -> vector registers"""
    if not os.path.exists(mq_build.LIB):
        pytest.fail(f"{mq_build.LIB} is not built (python -c 'import __graft_entry__ as g; g.build()')")
    if not (os.path.exists(OBJDUMP) and os.path.exists(READELF)):
        pytest.skip("no llvm-objdump and llvm-readelf")
    folder = tmp_path_factory.mktemp("lib")
    shutil.copy(mq_build.LIB, folder / "lib.so")
    subprocess.run([OBJDUMP, "--offloading", "lib.so"], cwd=folder, check=True, capture_output=True)
    out = {}
    for name in os.listdir(folder):
        if "gfx950" in name:
            notes = subprocess.run([READELF, "--notes", name], cwd=folder, check=True, capture_output=True, text=True).stdout
            for kernel in notes.split(".agpr_count")[1:]:
                out[re.search(r"\.name:\s+(\S+)", kernel).group(1)] = int(re.search(r"\.vgpr_count:\s+(\d+)", kernel).group(1))
    return out


def test_general_decode_kernel(registers):
    seen = 0
    for name, count in registers.items():
        m = re.match(r"_ZN2mq11gemv_kernelILi(\d)ELi(\d)ELi\dELi(\d+)EEE", name)
        if not m:
            continue
        r, row_groups, threads = map(int, m.groups())
        # (72000 rows take two row groups, 4096 one)
        plan = plans.gemv(4, 72000 if row_groups == 2 else 4096, 1024, r)
        assert plan.row_groups == row_groups
        roomy = plan.registers != 0
        assert (count <= 128) == (threads == 1024 or not roomy), (name, count, plan)
        seen += 1
    assert seen == 13


def test_kernels_that_sixteen_waves_share_a_compute_unit_with(registers):
    names = [n for n in registers if "gemv_quad_kernel" in n]
    assert len(names) == 48
    assert all(registers[n] <= 128 for n in names)

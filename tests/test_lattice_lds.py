"""What the restore kernels' LDS use has to keep to, by the compiler's figures.

The lattice walk reads its dynamic LDS from address 0, which holds while the
kernel has no LDS of its own (the library checks that too when it sets a
device up). The staged join's grid counts on four blocks per compute unit."""
import os
import re
import subprocess

import pytest

from paper_1803_11449_amd import build as lib_build

pytestmark = pytest.mark.slow


@pytest.fixture(scope="module")
def usage():
    """{kernel: {"LDS": bytes per block, "Occupancy": waves per SIMD}}"""
    if not os.path.exists(lib_build._hipcc()):
        pytest.skip("hipcc not installed")
    cmd = [lib_build._hipcc(), *lib_build.HIPCC_FLAGS, "--offload-device-only",
           "-Rpass-analysis=kernel-resource-usage", "-c",
           os.path.join(lib_build.CSRC, "restore.hip"), "-o", os.devnull]
    res = subprocess.run(cmd, capture_output=True, text=True)
    assert res.returncode == 0, res.stderr[-2000:]
    out, cur = {}, None
    for line in res.stderr.splitlines():
        m = re.search(r"remark: Function Name: (\S+)", line)
        if m:
            cur = out.setdefault(m.group(1), {})
        m = re.search(r"(LDS) Size \[bytes/block\]: (\d+)|(Occupancy) \[waves/SIMD\]: (\d+)", line)
        if m:
            cur[m.group(1) or m.group(3)] = int(m.group(2) or m.group(4))
    return out


def of(usage, name):
    return [v for n, v in usage.items() if f"{len(name)}{name}" in n]


def test_the_walk_has_no_static_lds(usage):
    assert [v["LDS"] for v in of(usage, "k_lattice")] == [0]
    assert of(usage, "k_scan_rows")[0]["LDS"] > 0               # the figure is read


def test_four_join_blocks_on_a_compute_unit(usage):
    """Of eight waves each: 8 waves per SIMD."""
    joins = of(usage, "k_join")
    assert len(joins) == 4
    assert all(v["LDS"] <= 163840 // 4 and v["Occupancy"] == 8 for v in joins), joins

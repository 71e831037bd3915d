"""What the restore kernels' resources have to keep to, by the compiler's figures.

The lattice walk reads its dynamic LDS from address 0, which holds while the
kernel has no LDS of its own (the library checks that too when it sets a
device up). The staged join's grid counts on four blocks per compute unit,
which the LDS and the scalar registers have to leave."""
import os
import re
import subprocess

import pytest

from paper_1803_11449_amd import build as lib_build

pytestmark = pytest.mark.slow


@pytest.fixture(scope="module")
def usage():
    """{kernel: {"LDS": bytes per block, "Occupancy": waves per SIMD, "SGPRs": number}}"""
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
        m = re.search(r"(LDS Size|Occupancy|TotalSGPRs)(?: \[[^]]*\])?: (\d+)", line)
        if m:
            cur[{"LDS Size": "LDS", "TotalSGPRs": "SGPRs"}.get(m.group(1), m.group(1))] = \
                int(m.group(2))
    return out


def of(usage, name):
    return [v for n, v in usage.items() if f"{len(name)}{name}" in n]


def test_the_walk_has_no_static_lds(usage):
    assert [v["LDS"] for v in of(usage, "k_lattice")] == [0]
    assert of(usage, "k_scan_rows")[0]["LDS"] > 0               # the figure is read


def test_four_join_blocks_on_a_compute_unit(usage):
    """Of eight waves each: 8 waves per SIMD, whose scalar registers (granules of
    16, and 16 more for the trap handler, which the compiler's occupancy leaves
    out) share 800."""
    joins = of(usage, "k_join")
    assert len(joins) == 4
    assert all(v["LDS"] <= 163840 // 4 and v["Occupancy"] == 8 for v in joins), joins
    assert all(8 * ((v["SGPRs"] + 15) // 16 * 16 + 16) <= 800 for v in joins), joins

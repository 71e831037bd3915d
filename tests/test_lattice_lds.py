"""The lattice walk reads its dynamic LDS from address 0, which holds while the
kernel has no LDS of its own: the compiler's figure for it is checked here,
and by the library when it sets a device up."""
import os
import re
import subprocess

import pytest

from paper_1803_11449_amd import build as lib_build

pytestmark = pytest.mark.slow


@pytest.mark.skipif(not os.path.exists(lib_build._hipcc()), reason="hipcc not installed")
def test_the_walk_has_no_static_lds():
    cmd = [lib_build._hipcc(), *lib_build.HIPCC_FLAGS, "--offload-device-only",
           "-Rpass-analysis=kernel-resource-usage", "-c",
           os.path.join(lib_build.CSRC, "restore.hip"), "-o", os.devnull]
    res = subprocess.run(cmd, capture_output=True, text=True)
    assert res.returncode == 0, res.stderr[-2000:]
    lds, cur = {}, None
    for line in res.stderr.splitlines():
        m = re.search(r"remark: Function Name: (\S+)", line)
        cur = m.group(1) if m else cur
        m = re.search(r"LDS Size \[bytes/block\]: (\d+)", line)
        if m:
            lds[cur] = int(m.group(1))
    sizes = {n: v for n, v in lds.items() if "k_lattice" in n or "k_scan_rows" in n}
    assert len(sizes) == 2 and all(v == 0 for n, v in sizes.items() if "k_lattice" in n), sizes
    assert all(v > 0 for n, v in sizes.items() if "k_scan_rows" in n)     # the figure is read

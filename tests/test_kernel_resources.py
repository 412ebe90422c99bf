"""Kernels whose arrays are meant to live in registers use no scratch memory,
from the compiler's own resource report (no GPU)."""
import os
import re
import subprocess

import pytest

from paper_2301_04835_amd import build

REPORTS = {}


def report(source):
    """{mangled kernel name: scratch bytes per lane} of one source."""
    if source not in REPORTS:
        r = subprocess.run([build.HIPCC] + build.FLAGS + ["--cuda-device-only", "-c", os.path.join(build.CSRC, source),
                            "-o", os.devnull, "-Rpass-analysis=kernel-resource-usage"],
                           capture_output=True, text=True)
        assert r.returncode == 0, r.stderr
        out, name = {}, None
        for line in r.stderr.splitlines():
            m = re.search(r"remark: +Function Name: (\S+)", line)
            name = m.group(1) if m else name
            m = re.search(r"remark: +ScratchSize \[bytes/lane\]: (\d+)", line)
            if m:
                out[name] = int(m.group(1))
        REPORTS[source] = out
    return REPORTS[source]


@pytest.mark.parametrize("source,kernel,instances", [("k_cell.hip", "k_cell_build", 4), ("k_grid.hip", "k_grid_step", 1),
                                                     ("k_grid.hip", "k_grid_step_wave", 1),
                                                     ("k_grid.hip", "k_grid_eval", 1)])
def test_no_scratch(source, kernel, instances):
    found = {k: v for k, v in report(source).items() if re.search(r"\d%s[IE]" % kernel, k)}
    assert len(found) == instances
    assert not any(found.values()), found

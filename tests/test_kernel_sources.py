"""What the kernels' helpers promise their callers, read from the sources."""
import os
import re

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2301_04835_amd", "csrc")


def test_workgroup_sum_frees_its_lds():
    """block_sum0 leaves through a barrier, so that a caller's loop may pass
    the same LDS again: thread 0 still reads it while the other wavefronts run
    ahead.  One definition, which every kernel includes."""
    found = []
    for f in sorted(os.listdir(CSRC)):
        with open(os.path.join(CSRC, f)) as fh:
            text = fh.read()
        for m in re.finditer(r"void block_sum0\(.*?\n}\n", text, re.S):
            found.append((f, m.group(0)))
    assert [f for f, _ in found] == ["dev_reduce.h"]
    assert found[0][1].endswith("    __syncthreads();\n}\n")

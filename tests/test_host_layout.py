"""CPU-side checks of what the host decides before a launch: how the kernels are built, and how large a step's workspace is."""
import glob
import os
import re

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def ff():
    import paper_2506_22771_amd as m
    try:
        m.lib()
    except FileNotFoundError:
        import __graft_entry__ as g
        g.build()
        m.lib()
    return m


def test_kernels_have_no_overridable_build_variants():
    """Every kernel is built in one form.  A switch that a -D option can flip is a kernel that no test runs: with two of them
    the three-stage pipeline missed a stage and the weight update of the contraction stored through a null pointer."""
    found = []
    for path in sorted(glob.glob(os.path.join(ROOT, "paper_2506_22771_amd", "csrc", "*"))):
        for n, line in enumerate(open(path), 1):
            if re.match(r"\s*#\s*(if|ifdef|ifndef|elif)\b", line):
                found.append(f"{os.path.basename(path)}:{n}: {line.strip()}")
    assert not found, found

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


def test_only_patch_matrices_that_are_read_again_are_kept_per_layer(ff):
    """A layer of more than four channels whose channel count is no multiple of four needs its patch matrix for the forward
    contraction only: one scratch serves all such layers of a step.  What a further layer adds to the workspace is its int8
    input, its accumulators and its per-sample words, not the patches (nine times the input)."""
    from workloads import Layer
    B, side, C = 32, 16, 18

    def bytes_of(k):
        layers = [Layer("conv", H=side, W=side, C_in=C, C_out=C, ksize=3, stride=1, pad=1) for _ in range(k)]
        descs = (ff.binding.LayerDesc * k)(*[ff.layer_desc(l, B) for l in layers])
        net = ff.binding.NetDesc(k, B, descs, None, 0, None, 1)
        return int(ff.lib().ff_workspace_bytes(ff.binding.C.byref(net)))

    M = B * side * side
    kept = 2 * M * ff.ff_pitch(C) + 2 * M * ff.ff_pitch32(C) * 4   # both passes
    words = 2 * B * (8 + 4 + 4 + 4) + 64                           # sums, maxima, two coefficients, scales
    patches = 2 * M * ff.ff_pitch(9 * C)
    assert patches > 2 * kept - 2 * M * ff.ff_pitch32(C) * 4       # (the bound below tells the two apart)
    for k in (2, 3, 6):
        assert bytes_of(k + 1) - bytes_of(k) <= kept + words + 16 * 256, k

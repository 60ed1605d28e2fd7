"""Which kernels the launch modes put to work: one per operation (every tensor in memory) in FF_LAUNCH_KERNELS, shared ones otherwise."""
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

from workloads import bottleneck_stack, res_stack  # noqa: E402


@pytest.fixture(scope="module")
def ff():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2506_22771_amd as m
    m.lib()
    return m


from graph_util import step_kernels  # noqa: E402


@pytest.mark.parametrize("mode,launches", [("kernels", 3), ("lanes", 0), ("auto", 0)])
def test_block_outputs_have_launches_of_their_own(ff, mode, launches):
    """Three blocks, maps of 256 and 64 pixels."""
    names = [n for n, _ in step_kernels(res_stack(16, [(16, 1, 2), (32, 2, 1)], 16, 16), 4, mode)]
    assert sum("k_residual_act" in n for n in names) == launches
    assert sum("k_goodness_fx" in n for n in names) == max(1, launches)   # (the last block's, in any mode)


@pytest.mark.parametrize("mode", ["kernels", "lanes", "auto"])
@pytest.mark.parametrize("B", [64, 256])   # 2^21 and 2^23 outputs of the depthwise layer
def test_accumulators_worked_out_again(ff, mode, B):
    """Stem, 1x1 expansion, depthwise layer and 1x1 projection: goodness sums, hand-off (not the last layer's) and local gradient."""
    names = [n for n, _ in step_kernels(bottleneck_stack(16, [(2, 24, 1)], 32, 32), B, mode)]
    depthwise = 3 if mode != "kernels" and B == 256 else 0
    assert sum("k_rows_i8" in n for n in names) == (0 if mode == "kernels" else 8)
    assert sum("k_dwconv_rework" in n for n in names) == depthwise
    assert sum("k_dwconv_forward" in n for n in names) == (0 if depthwise else 1)


@pytest.mark.parametrize("side,C,stride,reworked", [(32, 64, 1, True), (30, 96, 1, False), (32, 64, 2, False), (16, 144, 1, False)])
def test_depthwise_layers_worked_out_again(ff, side, C, stride, reworked):
    """Strips of whole groups of four pixels, and workgroups that are not half empty."""
    names = [n for n, _ in step_kernels(bottleneck_stack(C, [(1, 16, stride)], side, side), 256, "lanes")]
    assert any("k_dwconv_rework" in n for n in names) == reworked

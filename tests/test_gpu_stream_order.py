"""What the launches of a step wait for: the projection of a residual block runs beside the block's two convolutions, and whichever
launch forms the block output waits for both."""
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

from workloads import res_stack  # noqa: E402


@pytest.fixture(scope="module")
def ff():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2506_22771_amd as m
    m.lib()
    return m


from graph_util import step_kernels  # noqa: E402


@pytest.mark.parametrize("side,reader", [(12, "k_residual_act"),   # 36 rows a sample: a launch of its own forms the block output
                                         (16, "k_gemm_nt_i8")])    # 64: the contraction does
def test_projection_runs_beside_the_second_convolution(ff, side, reader):
    nodes = step_kernels(res_stack(16, [(32, 2, 1)], side, side), 5, "lanes")
    # in the forward pass one launch waits for two others: the one that reads the projection's accumulators
    joined = [(name, deps) for name, deps in nodes if len(deps) > 1 and not any("k_goodness" in d for d in deps)]
    assert len(joined) == 1 and reader in joined[0][0], nodes
    assert any("k_gemm_nt_i8" in d for d in joined[0][1])

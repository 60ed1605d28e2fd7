"""Residual blocks whose output is formed in the contraction and whose goodness sums are formed by the next layer's quantiser, against
the CPU oracle: tiles of whole, partial and several samples, row counts that are no multiple of four, identity and projection, a
dense reader, the last block (no reader)."""
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

from workloads import Layer, Workload, res_stack  # noqa: E402


@pytest.fixture(scope="module")
def ff():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2506_22771_amd as m
    m.lib()
    return m


from test_gpu_parity import _matched_thetas, _run_steps  # noqa: E402


@pytest.mark.parametrize("H,W,B,stem,stages,head", [
    (16, 16, 4, 16, [(16, 1, 2), (36, 2, 1)], 0),      # two tiles a sample, then samples of 64 rows
    (28, 28, 3, 32, [(32, 1, 1), (64, 2, 2)], 0),      # 784 and 196 rows
    (7, 9, 5, 16, [(16, 1, 1), (32, 2, 1)], 24),       # 63 rows, a dense reader of 20 x 32 features
    (5, 4, 9, 20, [(20, 1, 1), (20, 1, 1)], 0),        # 20 rows: six samples in a tile
    (8, 8, 17, 64, [(64, 1, 2)], 0)])                  # 64 rows, several blocks
@pytest.mark.parametrize("mode", ["auto", "kernels"])
def test_residual_step_block_outputs(ff, H, W, B, stem, stages, head, mode):
    layers = res_stack(stem, stages, H, W)
    if head:
        layers += (Layer("dense", in_features=layers[-1].H_out * layers[-1].W_out * layers[-1].C_out, out_features=head),)
    wl = Workload("res", layers, B, "normal", lam=0.05)
    _run_steps(ff, wl, 1, theta_layer=_matched_thetas(wl), launch_mode=mode)


def test_residual_step_with_resident_weights(ff):
    """Blocks large enough for the resident-weight contraction."""
    wl = Workload("res", res_stack(64, [(64, 1, 1)], 32, 32), 9, "normal", lam=0.05)
    _run_steps(ff, wl, 1, theta_layer=_matched_thetas(wl))

"""GPU parity at the sizes where a kernel's tiling, remainders or dispatch change: integer outputs bit for bit against the
CPU oracle."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

from oracle import ff_oracle as O  # noqa: E402
from workloads import Layer  # noqa: E402


@pytest.fixture(scope="module")
def ff():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2506_22771_amd as m
    m.lib()
    return m


from gpu_util import dev, empty32, pad8, pad_nhwc, workspace  # noqa: E402


@pytest.mark.parametrize("relu", [1, 0])
@pytest.mark.parametrize("B,H,W,Cin,Cout", [(70, 1, 1, 16, 24), (40, 1, 2, 16, 40), (9, 3, 5, 32, 72), (11, 7, 7, 16, 33),
                                            (5, 5, 13, 3, 130), (3, 28, 28, 1, 20), (37, 4, 4, 16, 64), (2, 31, 33, 16, 257)])
def test_conv_goodness_sums_of_any_map_size(ff, B, H, W, Cin, Cout, relu):
    """Per-sample sums and maxima where a 32-row tile holds whole, partial and several samples."""
    rng = np.random.default_rng(H * 100 + W)
    layer = Layer("conv", H=H, W=W, C_in=Cin, C_out=Cout, ksize=3, stride=1, pad=1, relu=relu)
    desc = ff.layer_desc(layer, B)
    a_q = rng.integers(-127, 128, (B, H, W, Cin)).astype(np.int8)
    w_q = rng.integers(-127, 128, (Cout, 3, 3, Cin)).astype(np.int8)
    acc_ref = O.conv_forward(a_q, w_q, 1, 1)
    g_ref = O.goodness(acc_ref, relu, O.goodness_shift(layer.K, layer.terms_per_sample), np.float32(0.01), np.float32(0.02))
    acc = empty32(B * H * W, Cout)
    gsum = torch.full((B,), 7, dtype=torch.int64, device="cuda")
    vmax = torch.full((B,), 9, dtype=torch.int32, device="cuda")
    ff.ff_layer_forward(desc, dev(pad_nhwc(a_q)), dev(pad8(w_q.reshape(Cout, -1))), acc, gsum, vmax,
                        workspace(ff.ff_layer_workspace_bytes(desc)))
    torch.cuda.synchronize()
    np.testing.assert_array_equal(acc.cpu().numpy()[:, :Cout], acc_ref.reshape(-1, Cout))
    np.testing.assert_array_equal(gsum.cpu().numpy().view(np.uint64), g_ref["g_int"])
    np.testing.assert_array_equal(vmax.cpu().numpy(), g_ref["vmax"])

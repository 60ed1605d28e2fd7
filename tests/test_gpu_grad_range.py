"""Local gradients whose range the quantiser forms itself from the per-sample factors and maxima (small batches) or is handed
(larger ones), against the CPU oracle: the largest gradient in the first, a middle and the last sample."""
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


from gpu_util import check_q, dev, empty32, empty8, pad32, pad8, scalar, workspace  # noqa: E402


@pytest.mark.parametrize("B", [1, 255, 1025, 2047, 2048, 2049])
@pytest.mark.parametrize("where", [0.0, 0.5, 1.0])
def test_gradient_range_of_a_batch(ff, B, where):
    rng = np.random.default_rng(B)
    N, K = 24, 20
    desc = ff.layer_desc(Layer("dense", in_features=K, out_features=N), B)
    acc = rng.integers(-90000, 90000, (B, N)).astype(np.int32)
    ct = (rng.standard_normal(B) * 0.01).astype(np.float32)
    ct[int(where * (B - 1))] = np.float32(-0.7)
    s_a, s_w = np.float32(0.004), np.float32(0.0009)
    vmax = O.goodness(acc, 1, 0, s_a, s_w)["vmax"]
    q_ref, s_ref = O.quantize(O.local_grad(acc, 1, s_a, s_w, ct), 1, 4, 60)
    a_q = rng.integers(-127, 128, (B, K)).astype(np.int8)
    gy, s_g, dw = empty8(N, B), scalar(), empty32(N, K)
    ff.ff_layer_backward_local(desc, dev(pad32(acc)), dev(vmax), dev(np.array([s_a])), dev(np.array([s_w])), dev(ct), 1, 4, 60,
                               dev(pad8(a_q.T)), gy, s_g, dw, workspace(ff.ff_layer_workspace_bytes(desc)))
    torch.cuda.synchronize()
    assert s_g.item() == s_ref
    check_q(gy, q_ref.T, "gradient codes")

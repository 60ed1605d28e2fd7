"""Dense contractions with few outputs: tiles of 32 x 32 whose reduction four wavefronts share.  Remainders of tiles, of reduction steps
and of the wavefronts' shares; the limits of the rule that chooses the kernel."""
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


from gpu_util import dev, empty32, pad8, workspace  # noqa: E402
from graph_util import kernel_nodes  # noqa: E402


@pytest.mark.parametrize("B,K,N,relu,few", [
    (1, 1, 1, 1, True),
    (32, 128, 32, 1, True),       # one whole tile, one step: three wavefronts without work
    (33, 129, 31, 0, True),       # a second step of one byte, a second tile of one row
    (31, 512, 65, 1, True),       # a step for every wavefront
    (64, 513, 36, 1, True),       # one wavefront takes two
    (200, 1537, 500, 1, True),    # four steps for one wavefront, three for the others
    (95, 4704, 10, 0, True),
    (512, 300, 1024, 1, True),    # the most tiles
    (513, 300, 1024, 1, False),
    (20, 700, 1404, 1, False),    # more tiles a row than the reduction pays for
    (20, 704, 1404, 1, True)])
def test_forward_of_few_tiles(ff, B, K, N, relu, few):
    rng = np.random.default_rng(B + K + N)
    a_q = rng.integers(-127, 128, (B, K)).astype(np.int8)
    w_q = rng.integers(-127, 128, (N, K)).astype(np.int8)
    desc = ff.layer_desc(Layer("dense", in_features=K, out_features=N, relu=relu), B)
    acc_ref = O.dense_forward(a_q, w_q)
    g_ref = O.goodness(acc_ref, relu, O.goodness_shift(K, N), 0.01, 0.02)
    acc = empty32(B, N)
    gsum = torch.full((B,), 7, dtype=torch.int64, device="cuda")
    vmax = torch.full((B,), 9, dtype=torch.int32, device="cuda")
    d_a, d_w, ws = dev(pad8(a_q)), dev(pad8(w_q)), workspace()

    def forward():
        ff.ff_layer_forward(desc, d_a, d_w, acc, gsum, vmax, ws)

    assert any("k_few_nt_i8" in n for n, _ in kernel_nodes(forward)) == few
    forward()
    torch.cuda.synchronize()
    np.testing.assert_array_equal(acc.cpu().numpy()[:, :N], acc_ref)
    np.testing.assert_array_equal(gsum.cpu().numpy().view(np.uint64), g_ref["g_int"])
    np.testing.assert_array_equal(vmax.cpu().numpy(), g_ref["vmax"])


@pytest.mark.parametrize("B,K,N", [(3, 40, 1), (70, 33, 129), (129, 1000, 520), (40, 2000, 260)])
def test_input_gradient_of_few_tiles(ff, B, K, N):
    rng = np.random.default_rng(B + K + N)
    h_q = rng.integers(-127, 128, (B, N)).astype(np.int8)
    w_q = rng.integers(-127, 128, (N, K)).astype(np.int8)
    desc = ff.layer_desc(Layer("dense", in_features=K, out_features=N), B)
    e, ws = empty32(B, K), workspace()
    d_h, d_w = dev(pad8(h_q)), dev(pad8(np.ascontiguousarray(w_q.T)))

    def gradient():
        ff.ff_layer_input_grad(desc, d_h, d_w, e, ws)

    assert any("k_few_nt_i8" in n for n, _ in kernel_nodes(gradient))
    gradient()
    torch.cuda.synchronize()
    np.testing.assert_array_equal(e.cpu().numpy()[:, :K], O.dense_input_grad(h_q, w_q))

"""Forward contraction of 3x3 stride-1 convolutions with resident weights, and with streamed ones beyond 64 input channels: windows that
cross images and the ends of the tensor, odd widths, channel counts with half-empty pieces, ragged column blocks, tiles that end inside a
pass."""
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
from graph_util import kernel_nodes  # noqa: E402


@pytest.mark.parametrize("B,H,W,Cin,Cout,relu", [
    (16, 32, 32, 64, 64, 1),      # whole tiles of whole samples
    (3, 41, 29, 16, 260, 1),      # one piece a pixel, half of it empty; nine narrow column blocks, the last nearly empty
    (2, 30, 75, 32, 256, 0),      # a wide map: the widest windows; plain activations
    (5, 33, 31, 40, 228, 1),      # three chunks a pixel of which the last is half pad channels
    (9, 16, 16, 20, 512, 1),      # two chunks, the last a quarter full; eight column blocks
    (16, 12, 11, 64, 512, 1),     # samples of 132 rows
    (65, 16, 8, 8, 100, 1),       # 128 rows: two samples per tile; eight channels
    (70, 16, 16, 60, 36, 0)])     # one column block that is half empty
def test_conv_forward_with_resident_weights(ff, B, H, W, Cin, Cout, relu):
    rng = np.random.default_rng(B * W + Cin)
    layer = Layer("conv", H=H, W=W, C_in=Cin, C_out=Cout, ksize=3, stride=1, pad=1, relu=relu)
    desc = ff.layer_desc(layer, B)
    M, K = B * H * W, 9 * Cin
    a_q = rng.integers(-127, 128, (B, H, W, Cin)).astype(np.int8)
    w_q = rng.integers(-127, 128, (Cout, 3, 3, Cin)).astype(np.int8)
    acc = O.conv_forward(a_q, w_q, 1, 1).reshape(M, Cout)
    gd = O.goodness(acc.reshape(B, H * W * Cout), relu, O.goodness_shift(K, layer.terms_per_sample), np.float32(1), np.float32(1))
    d_acc = empty32(M, Cout)
    gsum = torch.full((B,), 7, dtype=torch.int64, device="cuda")
    vmax = torch.full((B,), 7, dtype=torch.int32, device="cuda")
    ws = workspace(ff.ff_layer_workspace_bytes(desc))
    d_a, d_w = dev(pad_nhwc(a_q)), dev(pad8(w_q.reshape(Cout, K)))

    def forward():
        ff.ff_layer_forward(desc, d_a, d_w, d_acc, gsum, vmax, ws)

    assert any("k_conv3_i8" in n for n, _ in kernel_nodes(forward))
    forward()
    torch.cuda.synchronize()
    np.testing.assert_array_equal(d_acc.cpu().numpy()[:, :Cout], acc)
    np.testing.assert_array_equal(gsum.cpu().numpy().view(np.uint64), gd["g_int"])
    np.testing.assert_array_equal(vmax.cpu().numpy(), gd["vmax"])


@pytest.mark.parametrize("B,H,W,Cin,Cout,relu,streamed", [
    (64, 32, 32, 128, 128, 1, True),    # whole tiles of 256 pixels, one a workgroup
    (600, 16, 16, 100, 132, 1, True),   # two tiles a workgroup; a second group of 36 channels, a second column block of four columns
    (700, 15, 17, 96, 68, 0, True),     # several tiles a workgroup, the last not full; plain activations
    (300, 29, 9, 108, 260, 1, True),    # channels that are no multiple of eight
    (1100, 8, 8, 128, 512, 1, True),    # four samples per tile
    (160, 13, 43, 192, 72, 1, True),    # a wide map: seven copies a window
    (20, 5, 70, 128, 80, 1, True),      # a wider one: 128-pixel tiles of six copies
    (3, 12, 11, 300, 68, 1, True),      # small: 128-pixel tiles, the second of a sample nearly empty
    (40, 4, 4, 512, 192, 1, True),      # eight samples per tile
    (2, 7, 7, 65 * 4, 76, 0, True),     # one tile that is not full
    (5, 3, 2, 288, 68, 1, True),
    # the limits of the rule: few channels and outputs, small maps, rounds that are not full, windows that do not fit
    (3, 12, 11, 100, 68, 1, False), (5, 3, 2, 96, 68, 1, False),
    (9, 18, 16, 128, 200, 0, False), (10, 18, 16, 128, 200, 0, True),
    (33, 14, 14, 96, 160, 1, False), (35, 14, 14, 96, 160, 1, True),
    (14, 8, 8, 256, 204, 1, False), (16, 8, 8, 256, 204, 1, True),
    (330, 7, 7, 192, 128, 1, False), (340, 7, 7, 192, 128, 1, True),
    (760, 8, 8, 128, 128, 1, False), (770, 8, 8, 128, 128, 1, True),
    (1030, 9, 12, 96, 128, 1, False), (1030, 9, 12, 100, 128, 1, True),
    (867, 5, 5, 112, 320, 1, False), (2, 9, 30, 192, 200, 1, True),
    (159, 5, 80, 128, 328, 1, True), (160, 5, 80, 128, 328, 1, False)])
def test_conv_forward_with_streamed_weights(ff, B, H, W, Cin, Cout, relu, streamed):
    rng = np.random.default_rng(B * W + Cin)
    layer = Layer("conv", H=H, W=W, C_in=Cin, C_out=Cout, ksize=3, stride=1, pad=1, relu=relu)
    desc = ff.layer_desc(layer, B)
    M, K = B * H * W, 9 * Cin
    a_q = rng.integers(-127, 128, (B, H, W, Cin)).astype(np.int8)
    w_q = rng.integers(-127, 128, (Cout, 3, 3, Cin)).astype(np.int8)
    d_acc = empty32(M, Cout)
    gsum = torch.full((B,), 7, dtype=torch.int64, device="cuda")
    vmax = torch.full((B,), 7, dtype=torch.int32, device="cuda")
    ws = workspace(ff.ff_layer_workspace_bytes(desc))
    d_a, d_w = dev(pad_nhwc(a_q)), dev(pad8(w_q.reshape(Cout, K)))

    def forward():
        ff.ff_layer_forward(desc, d_a, d_w, d_acc, gsum, vmax, ws)

    assert any("k_conv3_wide_i8" in n for n, _ in kernel_nodes(forward)) == streamed
    forward()
    torch.cuda.synchronize()
    # float64 sums of products below 2^31 are exact
    x = torch.nn.functional.pad(dev(a_q).double(), (0, 0, 1, 1, 1, 1))
    w = dev(w_q).double()
    acc = sum(x[:, kh:kh + H, kw:kw + W].reshape(M, Cin) @ w[:, kh, kw].t().contiguous() for kh in range(3) for kw in range(3))
    acc = acc.cpu().numpy().astype(np.int32)
    gd = O.goodness(acc.reshape(B, H * W * Cout), relu, O.goodness_shift(K, layer.terms_per_sample), np.float32(1), np.float32(1))
    np.testing.assert_array_equal(d_acc.cpu().numpy()[:, :Cout], acc)
    np.testing.assert_array_equal(gsum.cpu().numpy().view(np.uint64), gd["g_int"])
    np.testing.assert_array_equal(vmax.cpu().numpy(), gd["vmax"])

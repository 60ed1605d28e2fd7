"""Weight gradient of 3x3 convolutions from one input window per step: maps whose rows and images end
anywhere in a step, channel counts that leave tiles and 16-byte chunks partly empty, several sample chunks, single steps."""
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


from gpu_util import check_q, dev, empty8, pad32, pad_nhwc, scalar, workspace  # noqa: E402
from graph_util import kernel_nodes  # noqa: E402


@pytest.mark.parametrize("B,H,W,Cin,Cout", [
    (16, 32, 32, 64, 64),       # whole tiles, one step a workgroup
    (160, 32, 32, 32, 72),      # two sample chunks of different lengths, in two launches; a second tile of eight rows
    (256, 32, 32, 16, 64),      # two equal chunks in one launch; half a tile of input channels
    (15, 41, 29, 40, 130),      # rows end anywhere; three chunks a pixel, the last half pad channels; a reduction no multiple of 16
    (13, 9, 150, 33, 20),       # a wide map; channels that are no multiple of four
    (340, 7, 7, 96, 65),        # many images per step
    (1030, 4, 4, 128, 64),
    (1900, 3, 3, 16, 64),       # nearly as many zeros as pixels
    (130, 4, 4, 512, 500),      # tiles for half the chip, two steps, no split
    (2, 6, 2, 767, 1023)])      # one step, not filled
def test_conv_weight_gradient_from_windows(ff, B, H, W, Cin, Cout):
    rng = np.random.default_rng(B * W + Cin)
    layer = Layer("conv", H=H, W=W, C_in=Cin, C_out=Cout, ksize=3, stride=1, pad=1)
    desc = ff.layer_desc(layer, B)
    M, K, n_chunks = B * H * W, 9 * Cin, ff.ff_layer_dw_chunks(desc)
    a_q = rng.integers(-127, 128, (B, H, W, Cin)).astype(np.int8)
    acc = rng.integers(-200000, 200000, (M, Cout)).astype(np.int32)
    vmax = np.maximum(acc, 0).reshape(B, -1).max(axis=1).astype(np.int32)
    s_a, s_w = np.float32(0.0041), np.float32(0.0007)
    ct = (rng.standard_normal(B) * 0.3).astype(np.float32)
    gq_ref, sg_ref = O.quantize(O.local_grad(acc.reshape(B, H, W, Cout), 1, s_a, s_w, ct), 1, 4, 55)
    gq_ref = gq_ref.reshape(M, Cout)
    gy_t, s_g = empty8(Cout, M), scalar()
    dw = torch.full((n_chunks, Cout, ff.ff_pitch32(K)), 0x5A5A5A5A, dtype=torch.int32, device="cuda")
    ws = workspace(ff.ff_layer_workspace_bytes(desc))
    ws.fill_(0x5A)
    args = [dev(pad32(acc)), dev(vmax), dev(np.array([s_a])), dev(np.array([s_w])), dev(ct), 1, 4, 55, dev(pad_nhwc(a_q)), gy_t, s_g, dw, ws]
    assert any("k_wgrad3_i8" in n for n, _ in kernel_nodes(lambda: ff.ff_layer_backward_local(desc, *args)))
    ff.ff_layer_backward_local(desc, *args)
    torch.cuda.synchronize()
    assert s_g.item() == sg_ref
    check_q(gy_t, gq_ref.T, "gy_q_t")
    # float64 sums of products below 2^31 are exact
    x = torch.nn.functional.pad(dev(a_q).double(), (0, 0, 1, 1, 1, 1))
    g = dev(gq_ref).double().t().contiguous()
    per = B if n_chunks == 1 else 1 << ((133144 // (H * W)).bit_length() - 1)   # samples of a chunk
    assert (B + per - 1) // per == n_chunks
    for c in range(n_chunks):
        rows = slice(c * per * H * W, min(B, (c + 1) * per) * H * W)
        ref = torch.stack([g[:, rows].contiguous() @ x[:, kh:kh + H, kw:kw + W].reshape(M, Cin)[rows]
                           for kh in range(3) for kw in range(3)], dim=1).reshape(Cout, K)
        np.testing.assert_array_equal(dw[c, :, :K].cpu().numpy(), ref.cpu().numpy().astype(np.int64), err_msg=f"chunk {c}")

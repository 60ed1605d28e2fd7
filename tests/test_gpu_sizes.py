"""GPU parity at the sizes where a kernel's tiling, remainders or dispatch change: integer outputs bit for bit against the
CPU oracle."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

from oracle import ff_oracle as O  # noqa: E402
from workloads import Layer, Workload, bottleneck_stack, conv_stack, mlp  # noqa: E402


@pytest.fixture(scope="module")
def ff():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2506_22771_amd as m
    m.lib()
    return m


from gpu_util import check_q, dev, empty32, empty8, pad32, pad8, pad_nhwc, scalar, workspace  # noqa: E402
from test_gpu_parity import _matched_thetas, _run_steps  # noqa: E402


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


@pytest.mark.parametrize("B,H,W,Cin,Cout,ks,stride", [
    (2, 9, 7, 1, 20, 3, 1), (3, 28, 28, 1, 32, 3, 1), (2, 8, 12, 2, 17, 3, 2), (2, 10, 6, 4, 64, 3, 1), (2, 7, 9, 5, 18, 3, 1),
    (3, 5, 5, 8, 24, 3, 2), (2, 6, 11, 12, 40, 3, 1), (2, 13, 5, 14, 9, 3, 1), (2, 14, 14, 20, 33, 3, 2), (3, 7, 7, 24, 130, 3, 1),
    (2, 5, 3, 40, 70, 3, 1), (1, 4, 4, 120, 260, 3, 1), (2, 9, 9, 16, 16, 3, 2), (5, 7, 5, 20, 30, 1, 2), (4, 3, 1, 36, 52, 1, 1),
    (1, 3, 3, 516, 20, 3, 1), (70, 1, 1, 16, 16, 3, 1), (9, 28, 28, 64, 64, 3, 1), (40, 16, 16, 32, 48, 3, 2),
    (300, 8, 8, 24, 96, 3, 1)])
def test_conv_channel_counts_map_sizes_and_strides(ff, B, H, W, Cin, Cout, ks, stride):
    """Forward and weight gradient over every operand route: patch matrices of one to four channels, channel counts that
    are no multiple of 16 or of 4, maps narrower than a 16-byte chunk and not a multiple of anything, split reductions."""
    rng = np.random.default_rng(B * 100 + Cin)
    layer = Layer("conv", H=H, W=W, C_in=Cin, C_out=Cout, ksize=ks, stride=stride, pad=ks // 2)
    desc = ff.layer_desc(layer, B)
    K, M = layer.K, B * layer.rows_per_sample
    a_q = rng.integers(-127, 128, (B, H, W, Cin)).astype(np.int8)
    w_q = rng.integers(-127, 128, (Cout, ks, ks, Cin)).astype(np.int8)
    s_a, s_w = np.float32(0.0041), np.float32(0.0007)
    acc_ref = O.conv_forward(a_q, w_q, stride, ks // 2)
    r = O.goodness_shift(K, layer.terms_per_sample)
    g_ref = O.goodness(acc_ref, 1, r, s_a, s_w)
    ws = workspace(ff.ff_layer_workspace_bytes(desc))
    d_aq, acc = dev(pad_nhwc(a_q)), empty32(M, Cout)
    gsum = torch.full((B,), 7, dtype=torch.int64, device="cuda")
    vmax = torch.full((B,), 9, dtype=torch.int32, device="cuda")
    ff.ff_layer_forward(desc, d_aq, dev(pad8(w_q.reshape(Cout, K))), acc, gsum, vmax, ws)
    torch.cuda.synchronize()
    np.testing.assert_array_equal(acc.cpu().numpy()[:, :Cout], acc_ref.reshape(M, Cout))
    np.testing.assert_array_equal(gsum.cpu().numpy().view(np.uint64), g_ref["g_int"])
    ct = (rng.standard_normal(B) * 0.3).astype(np.float32)
    gq_ref, sg_ref = O.quantize(O.local_grad(acc_ref, 1, s_a, s_w, ct), 1, 4, 55)
    dw_ref = O.conv_wgrad(gq_ref, a_q, ks, stride, ks // 2, 0, B)
    gy_t, s_g, dw = empty8(Cout, M), scalar(), empty32(Cout, K)
    ws.fill_(0x5A)
    ff.ff_layer_backward_local(desc, dev(pad32(acc_ref.reshape(M, Cout))), dev(g_ref["vmax"]), dev(np.array([s_a])),
                               dev(np.array([s_w])), dev(ct), 1, 4, 55, d_aq, gy_t, s_g, dw, ws)
    torch.cuda.synchronize()
    assert s_g.item() == sg_ref
    check_q(gy_t, gq_ref.reshape(M, Cout).T, "gy_q_t")
    np.testing.assert_array_equal(dw.cpu().numpy()[:, :K], dw_ref.reshape(Cout, K))


@pytest.mark.parametrize("l2", [0, 1])
@pytest.mark.parametrize("rps,N,B", [(1, 64, 128), (1, 67, 129), (2, 30, 70), (3, 132, 50), (5, 32, 60), (49, 96, 6), (130, 65, 3)])
def test_handoff_and_local_gradient_codes_over_rows_per_sample(ff, rps, N, B, l2):
    """Whole and partial quantiser tiles, ragged columns, rows of one, several and many per sample, against the oracle."""
    rng = np.random.default_rng(rps * 1000 + N)
    if rps == 1:
        layer = Layer("dense", in_features=40, out_features=N, l2norm_out=l2)
    else:
        layer = Layer("conv", H=1, W=rps, C_in=16, C_out=N, ksize=3, stride=1, pad=1, l2norm_out=l2)
    desc = ff.layer_desc(layer, B)
    M = B * rps
    acc = rng.integers(-200000, 200000, (M, N)).astype(np.int32)
    acc[:rps] = np.minimum(acc[:rps], 0)            # a sample whose activities are all zero
    s_a, s_w = np.float32(0.0041), np.float32(0.0007)
    r = O.goodness_shift(layer.K, layer.terms_per_sample)
    g = O.goodness(acc.reshape(B, rps * N), 1, r, s_a, s_w)
    a = O.handoff(acc.reshape(B, rps * N), 1, l2, s_a, s_w, g["G"]).reshape(M, N)
    q_ref, s_ref = O.quantize(a, 1, 3, 21)
    q, q_t, s = empty8(M, N), empty8(N, M), scalar()
    d_acc, d_sa, d_sw = dev(pad32(acc)), dev(np.array([s_a])), dev(np.array([s_w]))
    ff.ff_layer_handoff(desc, d_acc, d_sa, d_sw, dev(g["G"]), dev(np.array([np.abs(a).max()], np.float32)), 1, 3, 21, q, q_t, s)
    torch.cuda.synchronize()
    assert s.item() == s_ref
    check_q(q, q_ref, "hand-off codes")
    check_q(q_t, q_ref.T, "transposed hand-off codes")


@pytest.mark.parametrize("channels,side,B", [
    ([3, 16, 20], 32, 8),      # a few splits, summed by the update one thread per group
    ([3, 16, 20], 32, 40),     # many splits of small outputs: sixteen lanes per group
    ([3, 8, 10], 24, 256),     # two equal sample chunks in one launch, rows that are no multiple of four
    ([1, 16, 7], 32, 140),     # two chunks of different sizes, one launch each
    ([2, 12], 28, 11)])
def test_step_with_split_and_chunked_weight_gradients(ff, channels, side, B):
    wl = Workload("split", conv_stack(channels, side, side), B, "uniform_onehot", lam=0.05)
    _run_steps(ff, wl, 1, theta_layer=_matched_thetas(wl), live=True)


@pytest.mark.parametrize("widths,B", [([33, 37, 30, 41], 70), ([130, 257, 66], 300)])
def test_chain_step_with_ragged_widths(ff, widths, B):
    wl = Workload("chain", mlp(widths, False), B, "normal", lam=0.3)
    _run_steps(ff, wl, 2, lookahead="chain", theta_layer=_matched_thetas(wl))


@pytest.mark.parametrize("rows,cols", [(20000, 1001), (20001, 1000), (600001, 32), (530000, 20), (70, 24), (129, 31), (65, 68), (63, 1025)])
@pytest.mark.parametrize("mode", [0, 1])
def test_quantize_tile_sizes(ff, rows, cols, mode):
    """Tensors with few and with many quantiser tiles, narrow ones among them, whole and ragged columns."""
    rng = np.random.default_rng(rows + cols)
    x = rng.standard_normal((rows, cols), dtype=np.float32)
    q_ref, s_ref = O.quantize(x, mode, 5, 77)
    q, q_t, s = empty8(rows, cols), empty8(cols, rows), scalar()
    ff.ff_quantize(dev(x), rows, cols, mode, 5, 77, q, q_t, s, workspace())
    torch.cuda.synchronize()
    assert s.item() == s_ref
    check_q(q, q_ref, "q")
    check_q(q_t, q_ref.T, "q_t")


@pytest.mark.parametrize("B,l2,depth", [(1, True, 2), (63, True, 3), (65, False, 3), (1024, True, 3), (1025, True, 2), (2048, False, 3), (2049, False, 3), (4096, False, 2),
                                        (4097, False, 2), (6144, True, 2), (6145, True, 2), (12288, False, 2), (12289, False, 2),
                                        (16384, True, 2), (16385, True, 2), (130, False, 19)])
def test_step_goodness_after_the_forward_pass_or_per_layer(ff, B, l2, depth):
    """Batches on both sides of the line between one goodness / look-ahead launch and one launch per layer; more layers
    than a workgroup of the single launch takes at a time."""
    wl = Workload("g", mlp([20] + [24, 17] * (depth // 2) + [16] * (depth % 2), l2), B, "normal", lam=0.3)
    _run_steps(ff, wl, 2, theta_layer=_matched_thetas(wl), launch_mode="kernels")


@pytest.mark.parametrize("rows", [1, 255, 257, 1000003])
@pytest.mark.parametrize("cols", [1, 2, 3, 4])
@pytest.mark.parametrize("mode", [0, 1])
def test_quantize_few_columns_row_major_only(ff, rows, cols, mode):
    rng = np.random.default_rng(rows + cols)
    x = rng.standard_normal((rows, cols), dtype=np.float32)
    q_ref, s_ref = O.quantize(x, mode, 5, 77)
    q, s = empty8(rows, cols), scalar()
    ff.ff_quantize(dev(x), rows, cols, mode, 5, 77, q, None, s, workspace())
    torch.cuda.synchronize()
    assert s.item() == s_ref
    check_q(q, q_ref, "q")


@pytest.mark.parametrize("B,K,N,relu", [
    (140000, 20, 100, 1), (135000, 150, 101, 0), (131100, 260, 128, 1),   # 256 x 128 tiles: one, three and five short steps
    (70000, 300, 250, 1), (66000, 70, 256, 0), (33000, 64, 500, 1),       # 128 x 256 tiles
    (9000, 48, 144, 1), (9000, 48, 96, 1), (5000, 200, 320, 0)])          # short reductions, narrow last tiles
def test_forward_tiles_two_workgroups_per_compute_unit(ff, B, K, N, relu):
    """Several tiles per workgroup, a count that does not divide evenly, ragged rows and columns in the last ones."""
    rng = np.random.default_rng(B + K)
    layer = Layer("dense", in_features=K, out_features=N, relu=relu)
    desc = ff.layer_desc(layer, B)
    a_q = rng.integers(-127, 128, (B, K)).astype(np.int8)
    w_q = rng.integers(-127, 128, (N, K)).astype(np.int8)
    acc_ref = (a_q.astype(np.float32) @ w_q.astype(np.float32).T).astype(np.int32)   # exact: |sum| < 2^24
    g_ref = O.goodness(acc_ref, relu, O.goodness_shift(K, N), np.float32(0.01), np.float32(0.02))
    acc = empty32(B, N)
    gsum = torch.full((B,), 7, dtype=torch.int64, device="cuda")
    vmax = torch.full((B,), 9, dtype=torch.int32, device="cuda")
    ff.ff_layer_forward(desc, dev(pad8(a_q)), dev(pad8(w_q)), acc, gsum, vmax, workspace())
    torch.cuda.synchronize()
    np.testing.assert_array_equal(acc.cpu().numpy()[:, :N], acc_ref)
    np.testing.assert_array_equal(gsum.cpu().numpy().view(np.uint64), g_ref["g_int"])
    np.testing.assert_array_equal(vmax.cpu().numpy(), g_ref["vmax"])


@pytest.mark.parametrize("blocks,H,W,B", [
    ([(2, 16, 1), (3, 24, 2)], 10, 12, 20),     # strips that end inside a map, then a stride of two
    ([(5, 8, 1)], 9, 8, 33), ([(9, 16, 1)], 7, 7, 40),   # two channel groups; a width that is no multiple of four
    ([(1, 8, 1)], 32, 32, 140)])                # two sample chunks of different sizes
def test_depthwise_step_partial_results(ff, blocks, H, W, B):
    wl = Workload("dw", bottleneck_stack(16, blocks, H, W), B, "normal", lam=0.05)
    _run_steps(ff, wl, 1, theta_layer=_matched_thetas(wl), live=True)


@pytest.mark.parametrize("mode,widths,B,updates", [
    ("lanes", [132, 260, 64], 70, 0), ("lanes", [1000, 333, 96], 200, 1), ("lanes", [64, 1001, 500, 40], 33, 1), ("lanes", [516, 132, 68], 130, 0),
    ("kernels", [2004, 2101, 40], 40, 1), ("kernels", [2000, 2048, 2001], 140, 0)])
def test_dense_step_with_the_update_in_the_weight_gradient(ff, mode, widths, B, updates):
    """Reduction lengths of one, two and three steps, ragged output tiles; a layer of 333, 1001 or 2101 inputs keeps the update
    as a launch of its own.  Beside other chains any small layer takes this route, alone on the chip one of at least two
    tiles per compute unit: the update launches of a step are counted."""
    wl = Workload("upd", mlp(widths, False), B, "normal", lam=0.3)
    thetas = _matched_thetas(wl)
    ff.ff_timing_reset()
    ff.ff_timing_enable(True, ["update"])
    try:
        _run_steps(ff, wl, 2, theta_layer=thetas, launch_mode=mode)
        launches = ff.ff_timing_read(ff.KERNEL_CLASSES.index("update"))[1]
    finally:
        ff.ff_timing_enable(False)
        ff.ff_timing_reset()
    assert launches == 2 * updates


@pytest.mark.parametrize("channels,side,B", [([3, 18, 30, 22], 9, 20), ([2, 6, 6, 9], 14, 33), ([5, 7], 11, 12)])
def test_step_with_patch_matrices_in_one_scratch(ff, channels, side, B):
    """Several layers whose forward pass goes through a patch matrix: those of more than four channels share the scratch."""
    wl = Workload("patches", conv_stack(channels, side, side), B, "normal", lam=0.05)
    _run_steps(ff, wl, 1, theta_layer=_matched_thetas(wl), live=True)


@pytest.mark.parametrize("n", [1, 7, 8191, 8193, 2048 * 1024 + 5, 256 * 8192, 2 * 256 * 8192 - 3, 2 * 256 * 8192 + 8193, 12_000_001])
@pytest.mark.parametrize("skew", [0, 1, 3])
def test_absmax_finds_the_largest_element_wherever_it_is(ff, n, skew):
    """The range of a tensor of one and several trips per workgroup, from any 4-byte aligned address: the largest magnitude at
    the ends, on the borders of the spans and in the unaligned head and tail."""
    buf = torch.full((n + skew,), 0.25, dtype=torch.float32, device="cuda")
    x = buf[skew:]
    q, s, ws = empty8(1, n), scalar(), workspace()
    for at in sorted({0, 1, 2, 3, n // 2, 8191, 8192, 256 * 8192 - 1, 256 * 8192, 256 * 8192 + 1, n - 5, n - 2, n - 1}):
        if not 0 <= at < n:
            continue
        x[at] = -508.0
        ff.ff_quantize(x, 1, n, 0, 0, 0, q, None, s, ws)
        assert s.item() == 4.0, at
        x[at] = 0.25


@pytest.mark.parametrize("B,H,W,Cin,Cout", [
    (128, 32, 32, 576, 128), (64, 32, 32, 320, 352),   # 128 x 256 tiles, the last columns half empty, rows nearly full
    (64, 32, 32, 320, 351), (200, 28, 28, 288, 128),   # one row less; two launches, the second too short for wide tiles
    (16, 16, 16, 256, 256), (64, 16, 16, 250, 256), (60, 17, 15, 256, 255), (64, 16, 16, 520, 130),   # short reductions:
    (16, 18, 15, 64, 300), (33, 13, 11, 29, 100)])                                                    # smaller tiles
def test_weight_gradient_tiles_of_long_and_short_reductions(ff, B, H, W, Cin, Cout):
    """A 1x1 convolution's weight gradient is a plain product, formed here in float64 (exact: sums below 2^31)."""
    rng = np.random.default_rng(B + Cin)
    layer = Layer("conv", H=H, W=W, C_in=Cin, C_out=Cout, ksize=1, stride=1, pad=0)
    desc = ff.layer_desc(layer, B)
    M, n_chunks = B * H * W, ff.ff_layer_dw_chunks(desc)
    a_q = rng.integers(-127, 128, (M, Cin)).astype(np.int8)
    acc = rng.integers(-200000, 200000, (M, Cout)).astype(np.int32)
    vmax = np.maximum(acc, 0).reshape(B, -1).max(axis=1).astype(np.int32)
    s_a, s_w = np.float32(0.0041), np.float32(0.0007)
    ct = (rng.standard_normal(B) * 0.3).astype(np.float32)
    gq_ref, sg_ref = O.quantize(O.local_grad(acc.reshape(B, H, W, Cout), 1, s_a, s_w, ct), 1, 4, 55)
    gq_ref = gq_ref.reshape(M, Cout)
    gy_t, s_g = empty8(Cout, M), scalar()
    dw = torch.full((n_chunks, Cout, ff.ff_pitch32(Cin)), 0x5A5A5A5A, dtype=torch.int32, device="cuda")
    ws = workspace(ff.ff_layer_workspace_bytes(desc))
    ws.fill_(0x5A)
    ff.ff_layer_backward_local(desc, dev(pad32(acc)), dev(vmax), dev(np.array([s_a])), dev(np.array([s_w])), dev(ct), 1, 4, 55,
                               dev(pad8(a_q)), gy_t, s_g, dw, ws)
    torch.cuda.synchronize()
    assert s_g.item() == sg_ref
    check_q(gy_t, gq_ref.T, "gy_q_t")
    got = dw.cpu().numpy()[:, :, :Cin].astype(np.int64).sum(axis=0)
    ref = dev(gq_ref).double().t().contiguous() @ dev(a_q).double()
    np.testing.assert_array_equal(got, ref.cpu().numpy().astype(np.int64))


@pytest.mark.parametrize("widths,B", [
    ([300, 301, 260], 4200),          # two partial results, one group of four columns per thread; a row that ends inside a group
    ([130, 127, 64], 9000),           # eight, sixteen lanes per group
    ([520, 516], 8200)])              # four, on the other side of the line between the two
def test_dense_update_sums_the_partial_results(ff, widths, B):
    wl = Workload("parts", mlp(widths, False), B, "normal", lam=0.05)
    _run_steps(ff, wl, 1, theta_layer=_matched_thetas(wl), launch_mode="kernels")


@pytest.mark.parametrize("rows,N", [(33111, 224), (17001, 500), (16500, 510), (70003, 72), (130001, 66)])
def test_codes_of_large_matrices_with_partial_tiles(ff, rows, N):
    """Whole-size quantiser tiles over int32 sources: partial tiles at both edges, rows of the source and of the codes that do
    not start on cache lines, a number of tile rows that is no multiple of eight."""
    rng = np.random.default_rng(rows + N)
    desc = ff.layer_desc(Layer("dense", in_features=24, out_features=N), rows)
    acc = rng.integers(-200000, 200000, (rows, N)).astype(np.int32)
    s_a, s_w = np.float32(0.0041), np.float32(0.0007)
    g = O.goodness(acc, 1, O.goodness_shift(24, N), s_a, s_w)
    a = O.handoff(acc, 1, 0, s_a, s_w, g["G"])
    q_ref, s_ref = O.quantize(a, 1, 3, 21)
    q, q_t, s = empty8(rows, N), empty8(N, rows), scalar()
    d_acc, d_sa, d_sw = dev(pad32(acc)), dev(np.array([s_a])), dev(np.array([s_w]))
    ff.ff_layer_handoff(desc, d_acc, d_sa, d_sw, dev(g["G"]), dev(np.array([np.abs(a).max()], np.float32)), 1, 3, 21, q, q_t, s)
    torch.cuda.synchronize()
    assert s.item() == s_ref
    check_q(q, q_ref, "hand-off codes")
    check_q(q_t, q_ref.T, "transposed hand-off codes")
    ct = (rng.standard_normal(rows) * 0.3).astype(np.float32)
    gq_ref, sg_ref = O.quantize(O.local_grad(acc, 1, s_a, s_w, ct), 1, 4, 55)
    gy_t, s_g, dw = empty8(N, rows), scalar(), empty32(N, 24)
    a_q = rng.integers(-127, 128, (rows, 24)).astype(np.int8)
    ff.ff_layer_backward_local(desc, d_acc, dev(g["vmax"]), d_sa, d_sw, dev(ct), 1, 4, 55, dev(pad8(np.ascontiguousarray(a_q.T))), gy_t, s_g,
                               dw, workspace(ff.ff_layer_workspace_bytes(desc)))
    torch.cuda.synchronize()
    assert s_g.item() == sg_ref
    check_q(gy_t, gq_ref.T, "gy_q_t")


@pytest.mark.parametrize("mode,fused", [("auto", 1), ("fused", 1), ("kernels", 0), ("lanes", 0)])
def test_launch_mode_of_a_small_stack_is_the_one_asked_for(ff, mode, fused):
    """A stack that FF_LAUNCH_AUTO would run as one launch: the other modes issue their own kernels."""
    wl = Workload("mode", mlp([40, 36, 20], False), 30, "normal", lam=0.3)
    thetas = _matched_thetas(wl)
    ff.ff_timing_reset()
    ff.ff_timing_enable(True, ["fused"])
    try:
        _run_steps(ff, wl, 2, theta_layer=thetas, launch_mode=mode)
        launches = ff.ff_timing_read(ff.KERNEL_CLASSES.index("fused"))[1]
    finally:
        ff.ff_timing_enable(False)
        ff.ff_timing_reset()
    assert launches == 2 * fused

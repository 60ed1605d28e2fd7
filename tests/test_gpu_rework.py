"""Steps whose layers work their accumulators out again instead of storing them, against the CPU oracle: remainders of the row
and column blocks, every reduction length class, maps of any size, frozen layers, rectified and plain activations."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

from workloads import Layer, Workload  # noqa: E402


@pytest.fixture(scope="module")
def ff():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2506_22771_amd as m
    m.lib()
    return m


from test_gpu_parity import _matched_thetas, _run_steps  # noqa: E402


def _stack(H, W, C, ks, relu=1):
    """Convolutions of stride 1, ks[i] wide, over C[0] -> C[1] -> ... channels; ks 0: depthwise."""
    return tuple(Layer("conv" if k else "dwconv", H=H, W=W, C_in=a, C_out=b, ksize=k or 3, stride=1, pad=(k or 3) // 2, relu=relu)
                 for a, b, k in zip(C, C[1:], ks))


@pytest.mark.parametrize("H,W,B,C,ks", [
    (16, 16, 5, [3, 32, 64, 68], [3, 1, 1]),      # two rows of 128 per sample; two chunks of the reduction; a third column block
    (7, 7, 11, [1, 20, 36, 20], [3, 1, 1]),       # samples of 49 rows; columns that end inside a block
    (28, 28, 2, [1, 32, 24, 132], [3, 1, 1]),     # samples of 784 rows, five column blocks
    (1, 1, 130, [16, 24, 12], [1, 1]),            # a row per sample, two rows beyond a block
    (4, 8, 9, [4, 128, 72, 64], [3, 1, 1]),       # samples of 32 rows; the longest reduction
    (8, 16, 3, [12, 100, 100, 56], [1, 0, 1]),    # into and out of a depthwise layer; a sample per block
    (9, 5, 6, [2, 96, 512], [3, 1]),              # the widest row of codes
    (10, 12, 6, [8, 144, 144, 24], [1, 0, 1]),    # depthwise strips that end inside a map; several channels beyond a wavefront's
    (9, 7, 5, [16, 40, 40, 20], [1, 0, 1]),       # depthwise pixels one by one (an odd width), quads of pad channels
    (1, 4, 40, [24, 24, 12], [0, 1])])      # a depthwise first layer, one row of pixels
def test_step_without_stored_accumulators(ff, H, W, B, C, ks):
    wl = Workload("rework", _stack(H, W, C, ks), B, "normal", lam=0.05)
    _run_steps(ff, wl, 1, theta_layer=_matched_thetas(wl), live=True, launch_mode="lanes")


def test_step_without_stored_accumulators_forms(ff):
    """Plain activations (floating-point rounding), both signs of the row's factor inside a block, and an all-zero input."""
    wl = Workload("rework", _stack(6, 8, [3, 24, 40, 40], [3, 1, 0], relu=0), 9, "normal", lam=0.05)
    _run_steps(ff, wl, 1, theta_layer=_matched_thetas(wl))
    wl = Workload("rework", _stack(6, 7, [3, 24, 40, 40], [3, 1, 0]), 9, "normal", lam=-3.0)
    _run_steps(ff, wl, 1, theta_layer=_matched_thetas(wl))
    zero = np.zeros((9, 6, 7, 3), np.float32)
    _run_steps(ff, wl, 1, inputs=(zero, zero))


@pytest.mark.parametrize("train", [[0, 1, 1], [1, 0, 1], [1, 1, 0]])
def test_step_without_stored_accumulators_frozen(ff, train):
    """The same layers stored (one kernel per operation) and worked out again, with frozen ones among them."""
    from paper_2506_22771_amd import schedule
    layers, B = _stack(8, 8, [3, 32, 48, 40], [3, 1, 1]), 10
    out = []
    for mode in ("kernels", "lanes"):
        g = torch.Generator(device="cuda").manual_seed(3)
        w = [torch.rand((l.N, l.K), generator=g, device="cuda") * 0.4 - 0.2 for l in layers]
        x = [torch.randn((B, layers[0].in_elems_per_sample), generator=g, device="cuda") for _ in range(2)]
        st = schedule.TrainState.from_weights(layers, B, w)
        net = ff.Net(layers, B, st.w_master, st.w_q, st.s_w, launch_mode=mode, theta_layer=[40.0] * 3, train_layer=train)
        loss, good = torch.empty((3, 2), device="cuda"), torch.empty((3, 2, B), device="cuda")
        ws = torch.empty(net.workspace_bytes(), dtype=torch.uint8, device="cuda")
        for step in range(3):
            ff.ff_train_step(net, x[0], x[1], 2.0, 0.05, 1e-4, 5, step, loss, good, ws)
        torch.cuda.synchronize()
        out.append([t.cpu() for t in (loss, good, *st.w_master, *st.w_q, *st.s_w)])
    assert all(torch.equal(a, b) for a, b in zip(*out))


from graph_util import step_kernels  # noqa: E402


@pytest.mark.parametrize("H,W,B,C,ks,relu,lam", [
    (32, 32, 128, [8, 64, 64, 16], [1, 0, 1], 1, 0.05),       # 2^23 outputs exactly, whole strips, full workgroups
    (27, 28, 111, [8, 100, 100, 16], [1, 0, 1], 1, 0.05),     # strips that end inside a map, quads of pad channels, a part of a workgroup
    (5, 12, 547, [8, 256, 256, 8], [1, 0, 1], 1, 0.05),       # one strip of five rows, workgroups three quarters full
    (32, 32, 128, [64, 64, 16], [0, 1], 1, 0.05),             # a depthwise first layer
    (32, 32, 128, [8, 64, 64, 16], [1, 0, 1], 0, 0.05),       # plain activations: floating-point rounding
    (27, 28, 111, [8, 100, 100, 16], [1, 0, 1], 1, -3.0)])    # factors of both signs
def test_large_depthwise_layers_without_stored_accumulators(ff, H, W, B, C, ks, relu, lam):
    layers = _stack(H, W, C, ks, relu)
    assert sum("k_dwconv_rework" in n for n, _ in step_kernels(layers, B, "lanes")) == 3
    wl = Workload("rework", layers, B, "normal", lam=lam)
    _run_steps(ff, wl, 1, theta_layer=_matched_thetas(wl), launch_mode="lanes")


def test_longest_rows_without_stored_accumulators(ff):
    """Rows of 128 bytes into a column block and a half, samples of 45 rows."""
    layers = _stack(5, 9, [4, 128, 48, 32], [3, 1, 1])
    assert sum("k_rows_i8" in n for n, _ in step_kernels(layers, 13, "lanes")) == 8
    wl = Workload("rework", layers, 13, "normal", lam=0.05)
    _run_steps(ff, wl, 1, theta_layer=_matched_thetas(wl), live=True, launch_mode="lanes")


def _modes_agree(ff, layers, B, steps, replay=False):
    """Steps with one kernel per operation, and as the library chooses (replayed from a graph): the same state after each."""
    from paper_2506_22771_amd import schedule
    k, sides = len(layers), []
    for mode in ("kernels", "lanes"):
        g = torch.Generator(device="cuda").manual_seed(3)
        w = [(torch.rand((l.N, l.K), generator=g, device="cuda") * 2 - 1) * (6.0 / l.fan_in) ** 0.5 for l in layers]
        x = [torch.randn((B, layers[0].in_elems_per_sample), generator=g, device="cuda") for _ in range(2)]
        st = schedule.TrainState.from_weights(layers, B, w)
        net = ff.Net(layers, B, st.w_master, st.w_q, st.s_w, launch_mode=mode, theta_layer=[40.0] * k)
        loss, good = torch.empty((k, 2), device="cuda"), torch.empty((k, 2, B), device="cuda")
        ws = torch.empty(net.workspace_bytes(), dtype=torch.uint8, device="cuda")
        count = torch.zeros(1, dtype=torch.int64, device="cuda")
        sides.append((net, x, loss, good, ws, count, st))

    def eager(side, step):
        net, x, loss, good, ws = side[:5]
        ff.ff_train_step(net, x[0], x[1], 2.0, 0.05, 1e-4, 5, step, loss, good, ws)

    def counted(side):
        net, x, loss, good, ws, count = side[:6]
        ff.ff_train_step_at(net, x[0], x[1], 2.0, 0.05, 1e-4, 5, count, 1, loss, good, ws)

    graph = None
    for step in range(steps):
        eager(sides[0], step)
        if not replay:
            eager(sides[1], step)
        elif graph is None:   # (the library's streams come into being outside a capture)
            counted(sides[1])
            graph = torch.cuda.CUDAGraph()
            with torch.cuda.graph(graph):
                counted(sides[1])
        else:
            graph.replay()
        torch.cuda.synchronize()
        a, b = (torch.cat([t.reshape(-1).view(torch.uint8) for t in (s[2], s[3], *s[6].w_master, *s[6].w_q, *s[6].s_w)]) for s in sides)
        assert torch.equal(a, b), step
        torch.randn(256, 256, device="cuda").matmul(torch.randn(256, 256, device="cuda"))   # the program's own work in between


@pytest.mark.parametrize("B,side,K,N", [(256, 16, 128, 384),    # 3 x 2^23 outputs of rows of 128 bytes
                                        (100, 28, 96, 328)])   # 82 column quads, a ragged last block
def test_wide_short_rows_stored_and_not(ff, B, side, K, N):
    layers = _stack(side, side, [16, K, N, 24], [1, 1, 1])
    names = [n for n, _ in step_kernels(layers, B, "lanes")]
    assert sum("k_rows_i8" in n for n in names) >= 5
    _modes_agree(ff, layers, B, 2)


def test_steps_without_stored_accumulators_from_a_graph(ff):
    """The random streams' step number is read from device memory in every pass that works accumulators out again."""
    layers = _stack(32, 32, [3, 16, 64, 64, 16], [3, 1, 0, 1])
    names = [n for n, _ in step_kernels(layers, 128, "lanes")]
    assert sum("k_dwconv_rework" in n for n in names) == 3 and sum("k_rows_i8" in n for n in names) == 8
    _modes_agree(ff, layers, 128, 4, replay=True)

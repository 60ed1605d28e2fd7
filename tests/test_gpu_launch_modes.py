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


from graph_util import kernel_nodes  # noqa: E402


def _kernels(ff, layers, B, mode):
    from paper_2506_22771_amd import schedule
    g = torch.Generator(device="cuda").manual_seed(3)
    w = [torch.rand((l.N, l.K), generator=g, device="cuda") * 0.4 - 0.2 for l in layers]
    x = [torch.randn((B, layers[0].in_elems_per_sample), generator=g, device="cuda") for _ in range(2)]
    st = schedule.TrainState.from_weights(layers, B, w)
    net = ff.Net(layers, B, st.w_master, st.w_q, st.s_w, launch_mode=mode)
    loss, good = torch.empty((len(layers), 2), device="cuda"), torch.empty((len(layers), 2, B), device="cuda")
    ws = torch.empty(net.workspace_bytes(), dtype=torch.uint8, device="cuda")

    def step():
        ff.ff_train_step(net, x[0], x[1], 2.0, 0.05, 1e-4, 5, 0, loss, good, ws)

    step()
    torch.cuda.synchronize()
    return [name for name, _ in kernel_nodes(step)]


@pytest.mark.parametrize("mode,launches", [("kernels", 3), ("lanes", 0), ("auto", 0)])
def test_block_outputs_have_launches_of_their_own(ff, mode, launches):
    """Three blocks, maps of 256 and 64 pixels."""
    names = _kernels(ff, res_stack(16, [(16, 1, 2), (32, 2, 1)], 16, 16), 4, mode)
    assert sum("k_residual_act" in n for n in names) == launches
    assert sum("k_goodness_fx" in n for n in names) == max(1, launches)   # (the last block's, in any mode)


@pytest.mark.parametrize("mode,launches", [("kernels", 0), ("lanes", 3), ("auto", 3)])
def test_accumulators_worked_out_again(ff, mode, launches):
    """Stem, 1x1 expansion, depthwise layer and 1x1 projection: goodness sums, hand-off and local gradient each."""
    names = _kernels(ff, bottleneck_stack(16, [(2, 24, 1)], 8, 8), 4, mode)
    assert sum("k_rows_i8" in n for n in names) == max(0, 3 * launches - 1)   # (the last layer hands nothing on)
    assert sum("k_dwconv_rework" in n for n in names) == launches
    assert sum("k_dwconv_forward" in n for n in names) == (0 if launches else 1)

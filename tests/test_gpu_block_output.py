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


from graph_util import step_kernels  # noqa: E402


@pytest.mark.parametrize("H,W,B,stem,stages,blocks", [
    (31, 29, 11, 20, [(20, 1, 1)], 1),        # one piece a pixel, narrow ragged columns; 899 rows: slices of two samples, a partial last tile
    (15, 19, 30, 36, [(36, 1, 2)], 2),        # two pieces, wide columns of which 36 exist; 285 rows
    (32, 30, 36, 16, [(32, 2, 1)], 1),        # a projection; 240 rows
    (30, 26, 42, 24, [(56, 2, 1)], 1),        # a projection, two pieces; 195 rows, 64 tiles in all
    (16, 9, 60, 12, [(12, 1, 1)], 1)])        # 144 rows: hardly more than half a tile
def test_block_output_with_resident_weights(ff, H, W, B, stem, stages, blocks):
    layers = res_stack(stem, stages, H, W)
    names = [n for n, _ in step_kernels(layers, B)]
    assert not any("k_residual_act" in n for n in names)
    assert sum("k_conv3_i8ILi2E" in n or "k_conv3_i8<2" in n for n in names) == blocks   # (the form that makes the block output)
    wl = Workload("res", layers, B, "normal", lam=0.05)
    _run_steps(ff, wl, 1, theta_layer=_matched_thetas(wl))


@pytest.mark.parametrize("H,W,B,stem,stage,tile", [
    (15, 14, 313, 72, (72, 1, 1), "256, 128, 4, 1"),      # 210 rows a sample: slices of two, a partial last tile; columns end in the tile
    (16, 16, 256, 72, (72, 1, 1), "256, 128, 4, 1"),      # whole tiles
    (31, 33, 250, 24, (72, 2, 1), "256, 128, 4, 1"),      # a projection; 272 rows a sample
    (15, 14, 160, 136, (136, 1, 1), "128, 256, 2, 2"),
    (30, 28, 160, 24, (136, 2, 1), "128, 256, 2, 2"),
    (16, 16, 256, 136, (136, 1, 1), "256, 256, 4, 2"),    # two tiles a workgroup, whose first copies wait for the tile before
    (31, 33, 250, 24, (136, 2, 1), "256, 256, 4, 2")])
def test_block_output_of_wide_tiles(ff, H, W, B, stem, stage, tile):
    """The implicit contraction's tiles with 64 x 128 accumulators a wavefront."""
    layers = res_stack(stem, [stage], H, W)
    mangled = "k_gemm_nt_i8I" + "".join(f"Li{v}E" for v in tile.split(", ") + ["4", "1"])
    names = [n for n, _ in step_kernels(layers, B)]
    assert sum(mangled in n or f"k_gemm_nt_i8<{tile}, 4, 1" in n for n in names) == 1
    wl = Workload("res", layers, B, "normal", lam=0.05)
    _run_steps(ff, wl, 1, theta_layer=_matched_thetas(wl))


@pytest.mark.parametrize("H,W,B,stem,stage", [
    (8, 8, 9, 324, (324, 1, 1)),        # 64 rows a sample, the fewest; columns end behind four of a block
    (5, 13, 7, 300, (300, 1, 1)),       # 65 rows: nearly every wavefront has two samples
    (22, 12, 9, 24, (324, 2, 1)),       # 66 rows, a projection
    (14, 14, 30, 100, (100, 1, 1)),     # 196 rows, a second group of 36 channels and as many columns
    (15, 17, 20, 128, (128, 1, 1)),     # 255 rows
    (28, 28, 86, 24, (192, 2, 1)),      # tiles of 256 x 128, the last of a pass not full, half of the second column block; a projection
    (14, 14, 86, 192, (192, 1, 1)),
    (15, 17, 300, 128, (128, 1, 1)),    # two tiles a workgroup, the second in the other pass behind one that is not full
    (5, 66, 60, 128, (128, 1, 1)),      # a wide map: tiles of 128 x 64, two a workgroup
    (8, 56, 74, 128, (128, 1, 1))])     # windows of seven copies
def test_block_output_with_streamed_weights(ff, H, W, B, stem, stage):
    layers = res_stack(stem, [stage], H, W)
    names = [n for n, _ in step_kernels(layers, B)]
    assert sum("k_conv3_wide_i8ILi2E" in n or "k_conv3_wide_i8<2" in n for n in names) == 1   # (the form that makes the block output)
    wl = Workload("res", layers, B, "normal", lam=0.05)
    _run_steps(ff, wl, 1, theta_layer=_matched_thetas(wl))


@pytest.mark.parametrize("H,W,B,head,reader", [
    (7, 7, 38, 0, True),      # 49 rows: several samples in a tile, their sums meet in LDS row by row
    (5, 6, 513, 20, True),    # a dense reader whose last row of tiles lies beyond the tensor, in the pitch of its transposed copy
    (8, 8, 2048, 0, True),    # the largest batch whose next layer forms the sums,
    (8, 8, 2049, 0, False),   # and beyond it
    (2, 2, 12289, 0, False)])   # goodness layer by layer
def test_goodness_sums_of_block_outputs(ff, H, W, B, head, reader):
    layers = res_stack(8, [(8, 1, 1), (12, 1, 1)], H, W)
    if head:
        layers = res_stack(8, [(8, 1, 1)], H, W) + (Layer("dense", in_features=H * W * 8, out_features=head),)
    names = [n for n, _ in step_kernels(layers, B, "lanes")]
    blocks = 1 if head else 2
    assert sum("k_goodness_fx" in n for n in names) == (blocks - 1 if reader else blocks)
    wl = Workload("res", layers, B, "normal", lam=0.05)
    _run_steps(ff, wl, 1, theta_layer=_matched_thetas(wl), launch_mode="lanes")

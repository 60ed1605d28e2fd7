"""Stochastic rounding at the edge between two codes, against the oracle: every element lies where its own 24 random bits k decide, at
a fraction of (k - 1) / 2^24, k / 2^24 or (k + 1) / 2^24 above a code (a random value meets that edge once in 2^24 elements).  The range
is 127, so that the quantiser's factor is exactly one."""
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
from graph_util import kernel_nodes  # noqa: E402

SEED, TAG = 6, 77
FORMS = ("k_quantizeILi{}ELb1ELi{}ELi{}ELi{}E", "k_quantize<{}, true, {}, {}, {}>")   # source, loads, column blocks, blocks per thread


def bits24(n):
    """The random bits of elements 0 .. n - 1."""
    first = O.hash_u32(SEED, TAG, 0)

    def mix(v):
        v = v ^ v >> 16
        v = v * 0x7FEB352D & 0xFFFFFFFF
        v ^= v >> 15
        v = v * 0x846CA68B & 0xFFFFFFFF
        return v ^ v >> 16

    def unmix(v):
        v ^= v >> 16
        v = v * pow(0x846CA68B, -1, 1 << 32) & 0xFFFFFFFF
        v ^= v >> 15 ^ v >> 30
        v = v * pow(0x7FEB352D, -1, 1 << 32) & 0xFFFFFFFF
        return v ^ v >> 16

    h = mix(np.arange(n, dtype=np.uint64) ^ np.uint64(unmix(first)))
    for i in (0, 1, n // 2, n - 1):
        assert int(h[i]) == O.hash_u32(SEED, TAG, i)
    return (h >> np.uint64(8)).astype(np.int64)


def edges(n, rng, codes):
    """Fixed-point values (24 bits behind the point) at the edges above the given codes."""
    base = rng.choice(np.array(codes, np.int64), n)
    return (base << 24) + np.clip(bits24(n) + rng.integers(-1, 2, n), 0, (1 << 24) - 1)


@pytest.mark.parametrize("rows,cols,loads,blocks,per_thread", [
    (8195, 1028, 2, 16, 2),      # whole tiles and ragged ones: fixed point
    (262150, 32, 2, 8, 2),
    (100, 252, 2, 16, 1),        # half-size tiles: floating point
    (2051, 4099, 0, 16, 2)])     # element loads
def test_tensor(ff, rows, cols, loads, blocks, per_thread):
    rng = np.random.default_rng(rows)
    x = (edges(rows * cols, rng, [0, 0, 1, 2, 5, 60, 125, -1, -1, -2, -3, -9, -126]).astype(np.float64) * 2.0 ** -24).astype(np.float32)
    x[rows * cols // 2] = 127.0
    x = x.reshape(rows, cols)
    q_ref, s_ref = O.quantize(x, 1, SEED, TAG)
    d_x, q, q_t, s, ws = dev(x), empty8(rows, cols), empty8(cols, rows), scalar(), workspace()

    def call():
        ff.ff_quantize(d_x, rows, cols, ff.ROUND_STOCHASTIC, SEED, TAG, q, q_t, s, ws)

    names = [n for n, _ in kernel_nodes(call)]
    assert any(f.format(0, loads, blocks, per_thread) in n for f in FORMS for n in names), names
    call()
    torch.cuda.synchronize()
    assert s.item() == s_ref == 1.0
    check_q(q, q_ref, "codes")
    check_q(q_t, q_ref.T, "transposed codes")


def accumulators(rows, cols, rng, down):
    """Accumulators at the edges, of which an eighth is rectified away; down: rows whose factor is negative."""
    acc = edges(rows * cols, rng, [0, 0, 0, 1, 2, 9, 60, 125]).reshape(rows, cols)
    acc = np.where(down[:, None], (127 << 24) - acc, acc)   # (the fraction of -t is one minus that of t)
    acc = np.where(down[:, None] & (acc > 8 << 24) & (rng.random(acc.shape) < 0.7), acc & ((1 << 24) - 1), acc)   # (exact in fp32)
    acc = np.where(rng.random(acc.shape) < 0.125, -acc, acc)
    acc[rows // 2, cols // 2] = 127 << 24
    return acc.astype(np.int32)


@pytest.mark.parametrize("B,N", [(96, 256), (1030, 2052), (2500, 40), (70, 33)])
def test_local_gradient(ff, B, N):
    """Factors of -1 and 1."""
    rng = np.random.default_rng(B)
    K = 20
    ct = rng.choice(np.array([-0.5, 0.5], np.float32), B)
    acc = accumulators(B, N, rng, ct < 0)
    s = np.float32(2.0 ** -12)
    vmax = np.maximum(acc, 0).max(axis=1).astype(np.int32)
    q_ref, s_ref = O.quantize(O.local_grad(acc, 1, s, s, ct), 1, SEED, TAG)
    desc = ff.layer_desc(Layer("dense", in_features=K, out_features=N), B)
    a_q = rng.integers(-127, 128, (B, K)).astype(np.int8)
    gy, s_g, dw = empty8(N, B), scalar(), empty32(N, K)
    ff.ff_layer_backward_local(desc, dev(pad32(acc)), dev(vmax), dev(np.array([s])), dev(np.array([s])), dev(ct), 1, SEED, TAG,
                               dev(pad8(a_q.T)), gy, s_g, dw, workspace(ff.ff_layer_workspace_bytes(desc)))
    torch.cuda.synchronize()
    assert s_g.item() == s_ref == 1.0
    check_q(gy, q_ref.T, "gradient codes")


@pytest.mark.parametrize("B,N", [(96, 256), (1030, 2052), (70, 33)])
def test_handoff(ff, B, N):
    rng = np.random.default_rng(B)
    acc = accumulators(B, N, rng, np.zeros(B, bool))
    s = np.float32(2.0 ** -12)
    q_ref, s_ref = O.quantize(O.handoff(acc, 1, 0, s, s, np.ones(B, np.float32)), 1, SEED, TAG)
    desc = ff.layer_desc(Layer("dense", in_features=20, out_features=N), B)
    q, q_t, sc = empty8(B, N), empty8(N, B), scalar()
    ff.ff_layer_handoff(desc, dev(pad32(acc)), dev(np.array([s])), dev(np.array([s])), dev(np.ones(B, np.float32)),
                        dev(np.array([np.float32(127.0)])), 1, SEED, TAG, q, q_t, sc)
    torch.cuda.synchronize()
    assert sc.item() == s_ref == 1.0
    check_q(q, q_ref, "codes")
    check_q(q_t, q_ref.T, "transposed codes")

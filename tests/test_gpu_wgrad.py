"""The weight gradients of layers 2 and 3 where their chunks, rings and sums can
go wrong: the FP32 chains on snapshots of a few rows, and, against FP64 sums,
chunks of several steps (the row ring, the double buffer, the rows loaded two
steps ahead), chunks that cross a layer or an x tile or end mid-column, both x
tiles, both step heights on either side of their rule, axes shorter than the
taps; and the trainer's gradient on a snapshot with a partial z tile.

Bars: sums of whole rows exactly; FP32 sums 1e-5 (relative L2), as for every
layer; the trainer's blocks 1e-2, as in test_gpu_cnn.py."""
import numpy as np
import pytest

from oracle import cnn
from paper_0712_2247_amd import hslb, workloads

pytestmark = pytest.mark.gpu


def weight_gradient(layer, nx, ny, nz, zper, a, g):
    op = hslb.HSLB_CNN_DW2 if layer == 2 else hslb.HSLB_CNN_DW3
    out = hslb.hslb_cnn_op(op, nx, ny, nz, zper, workloads.cnn_init_weights(23), a, g)
    n = g.shape[0] * 32 * 125
    return np.asarray(out[:n], dtype=np.float64).reshape(g.shape[0], 32, 125), np.asarray(out[n:], dtype=np.float64)


@pytest.mark.parametrize("layer", [2, 3])
@pytest.mark.parametrize("shape", [(32, 8, 2), (64, 8, 8), (32, 4, 16), (128, 4, 3), (96, 8, 4)],
                         ids=lambda s: "x".join(map(str, s)))
def test_rows_of_a_small_snapshot_are_summed_apart(shape, layer):
    """On a snapshot of a few rows an FP32 chain covers one row and the rows meet in
    FP64: in every four rows of the gradient lie 2^26, 1, 1 and -2^26 (one node
    each), whose FP32 sum is 0 or 1 and whose FP64 sum is 2."""
    nx, ny, nz = shape
    print(f"case {shape} layer {layer}", flush=True)
    co = 32 if layer == 2 else 3
    a = np.zeros((32, nz, ny, nx), dtype=np.float32)
    g = np.zeros((co, nz, ny, nx), dtype=np.float32)
    a[..., 8] = 2.0 ** 12
    for row, v in enumerate((2.0 ** 14, 2.0 ** -12, 2.0 ** -12, -2.0 ** 14)):
        g[:, :, row::4, 8] = v
    dW, _ = weight_gradient(layer, nx, ny, nz, False, a, g)
    want = np.zeros((co, 32, 125))
    for t, (dz, _, dx) in enumerate(cnn.TAPS):
        if dx == 0:
            want[:, :, t] = 2.0 * (ny // 4) * max(0, nz - abs(dz))
    assert np.array_equal(dW, want)


PARITY = [  # nx, ny, nz, zper
    (32, 4, 1, False), (32, 4, 2, False), (64, 4, 2, True), (64, 16, 24, False), (64, 16, 28, True), (64, 16, 29, False),
    (32, 4, 113, False), (64, 48, 12, True), (64, 64, 24, False), (128, 16, 20, True), (96, 8, 30, False),
    (96, 16, 30, True), (160, 12, 9, False),
]


@pytest.mark.parametrize("case", PARITY, ids=lambda c: "-".join(map(str, c)))
def test_weight_gradients_over_many_steps(case):
    nx, ny, nz, zper = case
    shape = (nz, ny, nx)
    a = workloads.bf16_grid_values((32,) + shape, 0.5, 38)
    for layer, seed in ((2, 39), (3, 40)):
        print(f"case {case} layer {layer}", flush=True)
        g = workloads.bf16_grid_values((32 if layer == 2 else 3,) + shape, 1e-3, seed)
        dW, db = weight_gradient(layer, nx, ny, nz, zper, a, g)
        g64 = g.astype(np.float64)
        want = cnn.conv_weight_grad(a.astype(np.float64), g64, zper)
        assert np.linalg.norm(dW - want) <= 1e-5 * np.linalg.norm(want)
        wb = g64.reshape(g.shape[0], -1).sum(axis=1)
        assert np.linalg.norm(db - wb) <= 1e-5 * np.linalg.norm(wb)


@pytest.mark.parametrize("shape", [(13, 16, 64), (6, 20, 96)], ids=lambda s: "x".join(map(str, s)))
def test_trainer_gradient_on_a_partial_z_tile(shape):
    """Pre-activations are kept packed, with the 1 or 2 rows that the last z
    tile has: a value read from another node's place would move the gradients of
    layers 1 and 2 by their own size."""
    nz, ny, nx = shape
    print(f"case {shape}", flush=True)
    walls = 1
    rng = np.random.default_rng(71)
    eta = 0.25 * (1.0 + 0.2 * rng.uniform(-1, 1, shape))
    eta[:walls] = 0.0
    eta[nz - walls:] = 0.0
    target = (0.02 * rng.standard_normal((3,) + shape)).astype(np.float32).astype(np.float64)
    w = workloads.cnn_init_weights(24)
    tr = hslb.Trainer(eta.size, eta.size)
    k = tr.add_host(eta, target, walls, walls)
    tr.set_weights(w)
    _, got = tr.grad(k)
    c = cnn.forward(w.astype(np.float64), eta, zper=False)
    _, gout = cnn.loss_and_grad_out(c["out"], target, cnn.fluid_mask(nz, ny, nx, walls, walls))
    want, _ = cnn.backward(w.astype(np.float64), c, gout)
    o = 0
    for name, shp in cnn.SHAPES:
        m = int(np.prod(shp))
        e = np.linalg.norm(got[o:o + m] - want[o:o + m]) / np.linalg.norm(want[o:o + m])
        print(f"{name} {e:.2e}", flush=True)
        assert e <= 1e-2, name
        o += m

"""GELU' of the input gradients where its two terms cancel (z near -0.7518): the
error of Phi(z) + z phi(z) evaluated with erfcf and expf, against FP64.

The bound follows from the roundings of that form.  At the zero both terms are
0.2261; in units of 1e-8 the argument of erfc moves Phi by up to 1.8, erfcf by 1.5
(one unit in the last place), the square and expf move the Gaussian term by 0.4 and
1.8 (one unit), its two products by 1.2 + 0.5: 7.2 at the most, and as independent
uniform roundings sqrt(1.8^2 + 1.5^2 + 0.4^2 + 1.8^2 + 1.2^2 + 0.5^2) / sqrt(3) =
1.9 rms.  The stored bf16 adds up to 2^-9 of the value, at most 2^-9 / sqrt(3) rms."""
import numpy as np
import pytest

from oracle import cnn
from paper_0712_2247_amd import hslb

pytestmark = pytest.mark.gpu

FORM_MAX, FORM_RMS = 7.2e-8, 1.9e-8


@pytest.mark.parametrize("op", [hslb.HSLB_CNN_DX3, hslb.HSLB_CNN_DX2], ids=["dx3", "dx2"])
def test_gelu_derivative_at_its_zero(op):
    nx, ny, nz = 32, 8, 6
    n = nx * ny * nz
    # an input gradient of exactly 1: one channel of ones through the centre tap
    p = {k: np.zeros(shp) for k, shp in cnn.SHAPES}
    p["W3" if op == hslb.HSLB_CNN_DX3 else "W2"][0, :, 62] = 1.0
    w = cnn.flatten(p).astype(np.float32)
    g = np.zeros((3 if op == hslb.HSLB_CNN_DX3 else 32, nz, ny, nx), dtype=np.float32)
    g[0] = 1.0
    z = (-0.7517915 + 2e-5 * np.random.default_rng(5).uniform(-1, 1, (32, nz, ny, nx))).astype(np.float32)
    out = np.asarray(hslb.hslb_cnn_op(op, nx, ny, nz, True, w, g, z), dtype=np.float64).reshape(2, 32 * n)
    assert np.all(out[0] == 1.0)
    want = cnn.gelu_grad(z.astype(np.float64)).ravel()
    assert np.abs(want).max() < 2e-5
    err = np.abs(out[1] - want)
    print(f"max {err.max():.2e} rms {np.sqrt((err ** 2).mean()):.2e}", flush=True)
    assert np.all(err <= FORM_MAX + 2.0 ** -9 * np.abs(want))
    assert np.sqrt((err ** 2).mean()) <= np.sqrt(FORM_RMS ** 2 + (2.0 ** -18 * want ** 2).mean() / 3)

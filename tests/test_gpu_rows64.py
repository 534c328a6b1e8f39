"""Collisions on x-rows of 64 nodes whose lanes share x-neighbour reads: under a
solid mask (solid lanes stay in the exchange), with FP64 storage, and for
populations beyond the cache (the streaming instance), against the FP64 oracle.

Bars, as for every step: FP64 1e-12 (relative L2), FP32 storage 1e-5."""
import numpy as np
import pytest

import oracle
from paper_0712_2247_amd import hslb, workloads

pytestmark = pytest.mark.gpu

CASES = [  # ny, nz, sigma, walls, precision, mask: past the small-lattice rules
    (41, 20, 5, 3, "f32", True), (40, 30, 8, 4, "f64", True), (33, 36, 4, 0, "f64", False), (64, 112, 6, 3, "f64", False),
    (64, 220, 3, 2, "f32", False),
]


@pytest.mark.parametrize("case", CASES, ids=lambda c: "-".join(map(str, c)))
def test_rows_of_64(case):
    ny, nz, sigma, walls, precision, masked = case
    print(f"case {case}", flush=True)
    shape = (nz, ny, 64)
    nb = workloads.number_density(0.2, sigma)
    n, u = workloads.random_state(shape, nb, 0.02, 1e-3, seed=ny + nz, solid_lo=walls, solid_hi=walls)
    kw = dict(accel=(1e-5, 2e-6, 0.0), wall_lo=walls, wall_hi=walls)
    g = hslb.Sim(64, ny, nz, sigma, 0.9, precision=precision, **kw)
    o = oracle.Oracle(64, ny, nz, sigma=sigma, tau=0.9, **kw)
    if masked:
        m = np.zeros(shape, dtype=np.uint8)
        m[nz // 2 - 3:nz // 2 + 3, 4:11, 60:] = 1   # touches a row's end, so its exchange wraps onto a solid lane
        m[nz // 2, :, 30] = 1
        n, u = n * (m == 0), u * (m == 0)
        g.set_solid(m)
        o.set_solid(m)
    g.init(n, u)
    o.init(n, u)
    g.step(3)
    o.step(3)
    bar = 1e-12 if precision == "f64" else 1e-5
    (gn, gu), (on, ou) = g.moments(), o.moments()
    for a, b in ((gn, on), (gu, ou)):
        assert np.linalg.norm(a - b) <= bar * np.linalg.norm(b)
    g.close()

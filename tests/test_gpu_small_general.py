"""The general kernels on lattices that the small-lattice kernels take by default
(hslb_set_small_lattice): against the FP64 oracle over the shapes of the step
tests (whole x-rows per block, blocks dealt in y bands with a partial last chunk,
rows of every kind for the fused moments, solid masks), and bit for bit against
the small-lattice kernels, which sum in the same order.

Bars, as in the step tests: FP64 populations 1e-13 (relative L2); FP32 fields 1e-5
over 5 steps (a velocity that decays from its random start has no such relative
bar over long runs); between the two paths equality."""
import numpy as np
import pytest

import oracle
from paper_0712_2247_amd import hslb, workloads

from . import test_gpu_attraction, test_gpu_masks, test_gpu_parity

pytestmark = pytest.mark.gpu


def rel(a, b):
    return float(np.linalg.norm(a - b) / np.linalg.norm(b))


def advance(nx, ny, nz, sigma, walls, precision, n, u, steps, mask=None, small=False, period=None, graph=True, **kw):
    g = hslb.Sim(nx, ny, nz, sigma, 0.9, accel=(1e-5, 2e-6, 0.0), wall_lo=walls, wall_hi=walls, precision=precision, **kw)
    hslb.hslb_set_small_lattice(g.ctx, small)
    hslb.hslb_set_graph(g.ctx, graph)
    if period is not None:
        hslb.hslb_set_shift_period(g.ctx, period)
    if mask is not None:
        g.set_solid(mask)
    g.init(n, u)
    g.step(steps)
    f, m = g.get_populations(), g.moments()
    g.close()
    return f, m


def compare(nx, ny, nz, sigma, walls, precision, n, u, mask=None, steps=20):
    args = (nx, ny, nz, sigma, walls, precision, n, u, steps)
    f, (gn, gu) = advance(*args, mask=mask)
    fs, (sn, su) = advance(*args, mask=mask, small=True)
    assert np.array_equal(f, fs) and np.array_equal(gn, sn) and np.array_equal(gu, su)
    if precision == "f32" and steps > 5:
        return
    o = oracle.Oracle(nx, ny, nz, sigma=sigma, tau=0.9, accel=(1e-5, 2e-6, 0.0), wall_lo=walls, wall_hi=walls)
    if mask is not None:
        o.set_solid(mask)
    o.init(n, u)
    o.step(steps)
    if precision == "f64":
        assert rel(f, o.get_populations()) <= 1e-13
    else:
        on, ou = o.moments()
        assert rel(gn, on) <= 1e-5 and rel(gu, ou) <= 1e-5


@pytest.mark.parametrize("precision", ["f64", "f32"])
@pytest.mark.parametrize("case", test_gpu_parity.CASES + test_gpu_parity.ROW_CASES + test_gpu_parity.BAND_CASES,
                         ids=lambda c: "x".join(map(str, c)))
def test_steps(case, precision):
    nx, ny, nz, sigma, walls = case
    print(f"case {case} {precision}", flush=True)
    n, u = workloads.random_state((nz, ny, nx), workloads.number_density(0.2, sigma), 0.02, 1e-3, seed=sigma + 7 * nz,
                                  solid_lo=walls, solid_hi=walls)
    compare(nx, ny, nz, sigma, walls, precision, n, u)


# Rows for the fused moments and row sums: several rows per block and idle
# threads, ny no multiple of the rows per block, rows of more than 256 nodes, the
# longest that one block takes, and one past it (separate kernels).
MOMENT_ROWS = [(100, 13, 8, 5, 0), (72, 11, 12, 4, 2), (33, 7, 10, 3, 2), (257, 5, 8, 3, 0), (300, 10, 6, 8, 0),
               (511, 5, 6, 2, 1), (512, 6, 5, 4, 0), (513, 5, 6, 3, 1)]


@pytest.mark.parametrize("precision", ["f64", "f32"])
@pytest.mark.parametrize("case", MOMENT_ROWS, ids=lambda c: "x".join(map(str, c)))
def test_rows_of_the_fused_moments(case, precision):
    nx, ny, nz, sigma, walls = case
    print(f"case {case} {precision}", flush=True)
    n, u = workloads.random_state((nz, ny, nx), workloads.number_density(0.2, sigma), 0.02, 1e-3, seed=nx,
                                  solid_lo=walls, solid_hi=walls)
    compare(nx, ny, nz, sigma, walls, precision, n, u, steps=5)


@pytest.mark.parametrize("precision", ["f64", "f32"])
@pytest.mark.parametrize("case", test_gpu_masks.CASES + [(100, 12, 16, 5, 3, 0.05, 6), (64, 14, 18, 7, 4, 0.05, 7)],
                         ids=lambda c: "x".join(map(str, c[:5])))
def test_obstacles(case, precision):
    print(f"case {case} {precision}", flush=True)
    m, n, u = test_gpu_masks._obstacles(case)
    compare(*case[:5], precision, n, u, mask=m)


@pytest.mark.parametrize("graph", [True, False], ids=["graph", "launches"])
@pytest.mark.parametrize("shape", [(16, 16, 24, 4, 2), (24, 20, 30, 8, 4)], ids=lambda c: "x".join(map(str, c)))
def test_steps_over_a_refresh_of_the_reference_tables(shape, graph):
    """FP32 populations are kept relative to the layers' means; the step that
    moves those reads with one table and writes with another."""
    nx, ny, nz, sigma, walls = shape
    print(f"case {shape} {graph}", flush=True)
    n, u = workloads.random_state((nz, ny, nx), workloads.number_density(0.2, sigma), 0.05, 2e-3, seed=9, solid_lo=walls,
                                  solid_hi=walls)
    a = advance(*shape, "f32", n, u, 23, small=True, period=5, graph=graph)
    b = advance(*shape, "f32", n, u, 23, small=False, period=5, graph=graph)
    assert np.array_equal(a[0], b[0]) and np.array_equal(a[1][0], b[1][0]) and np.array_equal(a[1][1], b[1][1])


ATTRACTION = [  # nx, ny, nz, sigma, walls, range, mask: with and without the fields kernel, axes the range wraps over
    (16, 16, 20, 4, 0, 4.0, False), (13, 12, 16, 3, 2, 2.0, False), (6, 8, 9, 3, 0, 10.0, False),
    (24, 20, 30, 8, 4, 3.0, False), (32, 32, 24, 6, 0, 4.0, False), (16, 16, 12, 8, 0, 10.0, False),
    (12, 10, 18, 4, 2, 2.5, True), (20, 22, 24, 6, 3, 2.5, True), (64, 10, 20, 4, 2, 3.0, False),
]


@pytest.mark.parametrize("precision", ["f64", "f32"])
@pytest.mark.parametrize("case", ATTRACTION, ids=lambda c: "x".join(map(str, c)))
def test_attraction(case, precision):
    """Both ways bit for bit, and in FP64 against the oracle."""
    nx, ny, nz, sigma, walls, reach, masked = case
    print(f"case {case} {precision}", flush=True)
    n, u = workloads.random_state((nz, ny, nx), workloads.number_density(0.2, sigma), 0.05, 2e-3, seed=nx + nz,
                                  solid_lo=walls, solid_hi=walls)
    m = None
    if masked:
        m = np.zeros((nz, ny, nx), dtype=np.uint8)
        m[nz // 2 - 1:nz // 2 + 1, 2:5, 3:6] = 1
        n, u = n * (m == 0), u * (m == 0)
    kw = dict(att_eps=2e-3, att_range=reach)
    args = (nx, ny, nz, sigma, walls, precision, n, u, 12)
    f, (gn, gu) = advance(*args, mask=m, **kw)
    fs, (sn, su) = advance(*args, mask=m, small=True, **kw)
    assert np.array_equal(f, fs) and np.array_equal(gn, sn) and np.array_equal(gu, su)
    if precision == "f64":
        o = oracle.Oracle(nx, ny, nz, sigma=sigma, tau=0.9, accel=(1e-5, 2e-6, 0.0), wall_lo=walls, wall_hi=walls, **kw)
        if masked:
            o.set_solid(m)
        o.init(n, u)
        o.step(12)
        assert rel(f, o.get_populations()) <= 1e-13


@pytest.mark.parametrize("case", test_gpu_attraction.CASES, ids=lambda c: "x".join(map(str, c[:6])))
def test_attraction_on_the_general_kernels(case):
    """The attraction's step cases, at the bar they have there."""
    print(f"case {case}", flush=True)
    n, u = test_gpu_attraction._state(case, seed=12)
    g, o = test_gpu_attraction._pair(case, accel=(1e-5, 0.0, 0.0))
    hslb.hslb_set_small_lattice(g.ctx, False)
    g.init(n, u)
    o.init(n, u)
    g.step(30)
    o.step(30)
    assert rel(g.get_populations(), o.get_populations()) <= 1e-13


# Either side of the lines at which a lattice leaves the fields kernel (its blocks
# resident at once, nodes a block forms, waves of the grid) and the split collide.
RULE_EDGES = [(6, 6, 512, 4, 0), (6, 6, 513, 4, 0), (16, 16, 256, 3, 0), (16, 16, 216, 4, 0), (16, 16, 217, 4, 0),
              (12, 16, 30, 6, 3), (12, 17, 30, 6, 3), (10, 10, 400, 5, 0), (10, 10, 401, 5, 0), (18, 18, 192, 2, 1),
              (16, 16, 160, 8, 4), (16, 16, 161, 8, 4)]


@pytest.mark.parametrize("precision", ["f64", "f32"])
@pytest.mark.parametrize("case", RULE_EDGES, ids=lambda c: "x".join(map(str, c)))
def test_edges_of_the_rule(case, precision):
    """Bit for bit the general kernels, whichever way the lattice goes."""
    nx, ny, nz, sigma, walls = case
    print(f"case {case} {precision}", flush=True)
    n, u = workloads.random_state((nz, ny, nx), workloads.number_density(0.2, sigma), 0.02, 1e-3, seed=nz + sigma,
                                  solid_lo=walls, solid_hi=walls)
    a = advance(nx, ny, nz, sigma, walls, precision, n, u, 6)
    b = advance(nx, ny, nz, sigma, walls, precision, n, u, 6, small=True)
    assert np.array_equal(a[0], b[0]) and np.array_equal(a[1][0], b[1][0]) and np.array_equal(a[1][1], b[1][1])

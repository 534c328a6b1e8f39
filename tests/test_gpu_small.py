"""The kernels of small lattices (fields of a layer per block, collision split
over six waves, the force straight from (n, u)) against the FP64 oracle, at the
edges of their rules: a block of exactly 1536 nodes and one just past it, planes
that are no multiple of 64, periodic axes shorter than the halo, the largest
node counts, masks and the attraction.

Bars, as for every step: FP64 1e-12 (relative L2) over the run, FP32 storage
1e-5; the force 1e-13 of its largest value."""
import numpy as np
import pytest
import torch

import oracle
from paper_0712_2247_amd import hslb, workloads

pytestmark = pytest.mark.gpu


def rel(a, b):
    return float(np.linalg.norm(a - b) / np.linalg.norm(b))


STEP_CASES = [  # nx, ny, nz, sigma, walls, precision, attraction range, mask
    (8, 8, 24, 4, 2, "f64", 0, False), (16, 16, 12, 5, 3, "f64", 0, False), (16, 17, 12, 4, 2, "f64", 0, False),
    (9, 9, 30, 7, 4, "f32", 0, False), (10, 11, 5, 8, 0, "f64", 0, False), (5, 6, 3, 2, 0, "f64", 0, False),
    (16, 16, 20, 4, 0, "f64", 4.0, False), (13, 12, 16, 3, 2, "f32", 2.0, False), (12, 12, 20, 4, 2, "f64", 0, True),
    (12, 10, 18, 4, 2, "f64", 2.5, True), (15, 12, 16, 5, 3, "f32", 0, True), (16, 16, 128, 4, 0, "f64", 0, False),
    (32, 32, 64, 3, 2, "f64", 0, False), (32, 32, 40, 6, 3, "f32", 0, False), (24, 20, 30, 8, 4, "f64", 3.0, False),
]


@pytest.mark.parametrize("case", STEP_CASES, ids=lambda c: "-".join(map(str, c)))
def test_small_steps(case):
    nx, ny, nz, sigma, walls, precision, att, masked = case
    print(f"case {case}", flush=True)
    nb = workloads.number_density(0.2, sigma)
    n, u = workloads.random_state((nz, ny, nx), nb, 0.02, 1e-3, seed=nx * 7 + nz, solid_lo=walls, solid_hi=walls)
    kw = dict(accel=(1e-5, 2e-6, 0.0), wall_lo=walls, wall_hi=walls)
    if att:
        kw.update(att_eps=1e-3, att_range=att)
    g = hslb.Sim(nx, ny, nz, sigma, 0.9, precision=precision, **kw)
    o = oracle.Oracle(nx, ny, nz, sigma=sigma, tau=0.9, **kw)
    if masked:
        m = np.zeros((nz, ny, nx), dtype=np.uint8)
        m[nz // 2 - 1:nz // 2 + 1, 2:5, 3:6] = 1
        n, u = n * (m == 0), u * (m == 0)
        g.set_solid(m)
        o.set_solid(m)
    g.init(n, u)
    o.init(n, u)
    g.step(5)
    o.step(5)
    bar = 1e-12 if precision == "f64" else 1e-5
    (gn, gu), (on, ou) = g.moments(), o.moments()
    assert rel(gn, on) <= bar and rel(gu, ou) <= bar
    g.close()


FORCE_CASES = [  # nx, ny, nz, sigma, walls, with u
    (24, 20, 30, 8, 4, True), (40, 40, 12, 8, 0, True), (17, 31, 21, 5, 3, True), (12, 13, 4, 6, 0, False),
    (39, 23, 60, 3, 2, True), (10, 40, 9, 8, 4, False),
]


@pytest.mark.parametrize("case", FORCE_CASES, ids=lambda c: "-".join(map(str, c)))
def test_force_of_device_fields(case):
    nx, ny, nz, sigma, walls, with_u = case
    print(f"case {case}", flush=True)
    nb = workloads.number_density(0.25, sigma)
    n, u = workloads.random_state((nz, ny, nx), nb, 0.05, 3e-3, seed=nx + nz, solid_lo=walls, solid_hi=walls)
    n[:walls] = 7.0  # values on solid layers are ignored
    kw = dict(accel=(1e-5, -2e-6, 0.0), wall_lo=walls, wall_hi=walls)
    o = oracle.Oracle(nx, ny, nz, sigma=sigma, tau=0.9, **kw)
    o.init(n, u if with_u else None)
    want = o.force()
    dev = torch.device("cuda:0")
    n_d = torch.from_numpy(n.ravel()).to(dev)
    u_d = torch.from_numpy(u.ravel()).to(dev) if with_u else None
    F_d = torch.full((3 * n.size,), float("nan"), dtype=torch.float64, device=dev)
    p = hslb.make_params(nx, ny, nz, sigma, 0.9, **kw)
    hslb.hslb_force_noalloc(p, n_d.data_ptr(), u_d.data_ptr() if with_u else 0, F_d.data_ptr(),
                            torch.cuda.current_stream(dev).cuda_stream)
    got = F_d.cpu().numpy().reshape(want.shape)
    assert np.abs(got - want).max() <= 1e-13 * np.abs(want).max()


def test_force_captured_beside_calls_of_another_size():
    """A captured force call whose block takes 83 KiB of LDS, replayed after calls
    of a lattice that takes 75 KiB: each replay gives the eager call's force."""
    dev = torch.device("cuda:0")
    calls = []
    for nx, ny, nz, sigma, walls in ((24, 20, 30, 8, 4), (20, 20, 40, 8, 4)):
        n, u = workloads.random_state((nz, ny, nx), workloads.number_density(0.25, sigma), 0.05, 3e-3, seed=nx,
                                      solid_lo=walls, solid_hi=walls)
        p = hslb.make_params(nx, ny, nz, sigma, 0.9, accel=(1e-5, 0.0, 0.0), wall_lo=walls, wall_hi=walls)
        calls.append((p, torch.from_numpy(n.ravel()).to(dev), torch.from_numpy(u.ravel()).to(dev),
                      torch.zeros(3 * n.size, dtype=torch.float64, device=dev)))

    def force(k):
        p, n, u, F = calls[k]
        hslb.hslb_force_noalloc(p, n.data_ptr(), u.data_ptr(), F.data_ptr(), torch.cuda.current_stream(dev).cuda_stream)
        return F

    want = force(0).clone()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        force(0)
    for _ in range(3):
        force(1)
        calls[0][3].zero_()
        torch.cuda.synchronize(dev)
        graph.replay()
        torch.cuda.synchronize(dev)
        assert torch.equal(calls[0][3], want)

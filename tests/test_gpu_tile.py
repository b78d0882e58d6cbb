"""GPU tests of the resident-tile passes (the automatic choice for grids of up
to about six million cells): bit for bit equal to the float32 oracle over
sizes around the tiles' edges (one cell, one row, odd widths whose edge tiles
move column by column, even widths whose edges are mirrored vectors, one tile,
many tiles) and step counts that give one pass, odd and even pass depths and
passes of two depths."""
import numpy as np
import pytest
import torch

import oracle
import workloads as W

pytestmark = pytest.mark.gpu

SHAPES = [(1, 1), (2, 3), (1, 130), (131, 1), (31, 64), (65, 96), (96, 34), (130, 257), (200, 700),
          (511, 514), (777, 1301), (1024, 1024), (1500, 1502), (2300, 2298)]


def _t(a):
    return torch.from_numpy(a).cuda()


@pytest.mark.parametrize("bc", ["periodic", "zeroflux"])
@pytest.mark.parametrize("shape", SHAPES, ids=lambda s: "%dx%d" % s)
def test_tile_passes_bitwise(shape, bc):
    from paper_2102_10340_amd import Simulation
    R, C = shape
    g = W.gene(W.PAPER_DEFAULT_GENE) if bc == "periodic" else W.PLAIN_GENE
    x = W.uniform_x(R, C, R + C)
    sim = Simulation(_t(x), g, bc, tuned=False)
    assert sim.pass_config()["kind"] == 4
    u, v = oracle.init_state(x, 1.0)
    for T in (1, 2, 7, 16, 33):
        print(f"case tile {shape} {bc} T={T}", flush=True)
        sim.step(T)
        u, v = oracle.run(u, v, g, bc, T, "f32")
        got = sim.read_host()
        assert np.array_equal(got[0], u) and np.array_equal(got[1], v), T
    sim.close()


@pytest.mark.parametrize("bc", ["periodic", "zeroflux"])
@pytest.mark.parametrize("shape", [(3, 5), (130, 257), (512, 512), (1100, 1400)],
                         ids=lambda s: "%dx%d" % s)
def test_tile_passes_gray_scott_bitwise(shape, bc):
    from paper_2102_10340_amd import Simulation
    R, C = shape
    gs = dict(dt=0.5, F=0.037, k=0.06, Du=0.2, Dv=0.1)
    rng = np.random.default_rng(R)
    u = np.ones((R, C), np.float32)
    v = rng.uniform(0, 0.3, (R, C)).astype(np.float32)
    sim = Simulation.gray_scott(_t(u), _t(v), bc=bc, **gs)
    assert sim.pass_config()["kind"] == 4
    for T in (5, 27):
        print(f"case tile gray-scott {shape} {bc} T={T}", flush=True)
        sim.step(T)
        u, v = oracle.gs_run(u, v, gs, bc, T)
        got = sim.read_host()
        assert np.array_equal(got[0], u) and np.array_equal(got[1], v), T
    sim.close()


def test_streamed_kernel_takes_the_larger_grids():
    from paper_2102_10340_amd import Simulation
    sim = Simulation(torch.zeros((2500, 2500), device="cuda"), W.PLAIN_GENE, tuned=False)
    assert sim.pass_config()["kind"] == 2
    sim.close()


@pytest.mark.parametrize("shape", [(1, 1), (7, 9), (64, 130), (300, 257)], ids=lambda s: "%dx%d" % s)
def test_read_into_device_views(shape):
    """A device read copies both planes in one launch, also to destinations that
    are not 16-byte aligned, and leaves what lies beside them."""
    from paper_2102_10340_amd import Simulation
    R, C = shape
    x = W.uniform_x(R, C, 3)
    sim = Simulation(_t(x), W.PLAIN_GENE, tuned=False).step(3)
    want = sim.state().clone()
    for off in (0, 1, 4):
        buf = torch.full((2, R * C + 8), 7.0, device="cuda")
        u, v = (buf[k, off:off + R * C].view(R, C) for k in range(2))
        sim.read_into(u, v)
        assert torch.equal(u, want[0]) and torch.equal(v, want[1]), off
        assert torch.all(buf[:, :off] == 7.0) and torch.all(buf[:, off + R * C:] == 7.0), off
    got = sim.read()
    assert torch.equal(got[0], want[0]) and torch.equal(got[1], want[1])
    sim.close()

"""GPU tests of the streamed forward passes' strips and of the pairs of wavefronts
that run the 8-step, four-column ones: bit for bit equal to the float32 oracle
where strips end at a zero-flux side (one strip exactly, one column group more,
strips that fill the grid exactly or overlap by one group, the fewest rows that
take them and one row less), where a torus wraps inside a strip, at odd widths,
and for pairs of one, two and many rows, for plain, recording and batched
passes."""
import numpy as np
import pytest
import torch

import oracle
import workloads as W

pytestmark = pytest.mark.gpu

PASSES = [(1, 8), (1, 16), (2, 3), (2, 12), (4, 8), (4, 12)]


def _shapes(cpl, K):
    w = 64 * cpl
    wout = w - 2 * (-(-K // cpl) * cpl)
    return [(K + 3, w), (K + 4, w), (K + 4, w + cpl), (40, w + wout), (37, w + wout + cpl),
            (50, w + 2 * wout - cpl), (33, w - cpl), (29, w + wout + 1)]


def _t(a):
    return torch.from_numpy(a).cuda()


@pytest.mark.parametrize("bc", ["periodic", "zeroflux"])
@pytest.mark.parametrize("cpl,K", PASSES)
def test_streamed_strips_bitwise(cpl, K, bc):
    from paper_2102_10340_amd import Simulation
    g = W.gene(W.PAPER_DEFAULT_GENE) if bc == "periodic" else W.PLAIN_GENE
    for R, C in _shapes(cpl, K):
        x = W.uniform_x(R, C, R + C)
        sim = Simulation(_t(x), g, bc, tuned=False)
        for seg in (0, 1, 7):
            print(f"case strips {R}x{C} {bc} cpl={cpl} K={K} seg={seg}", flush=True)
            sim.set_kernel(2, K, cpl, seg)
            u, v = (a.copy() for a in sim.read_host())
            sim.step(2 * K + 1)
            u, v = oracle.run(u, v, g, bc, 2 * K + 1, "f32")
            got = sim.read_host()
            assert np.array_equal(got[0], u) and np.array_equal(got[1], v), (R, C, seg)
        sim.close()


@pytest.mark.parametrize("bc", ["periodic", "zeroflux"])
@pytest.mark.parametrize("cpl", [1, 2])
def test_recording_strips_bitwise(cpl, bc):
    from paper_2102_10340_amd import Simulation
    K, T, g = 8, 19, W.PLAIN_GENE
    for R, C in _shapes(cpl, K):
        x = W.uniform_x(R, C, R * C)
        print(f"case recording strips {R}x{C} {bc} cpl={cpl}", flush=True)
        want = [oracle.init_state(x, 1.0)]
        for _ in range(T):
            want.append(oracle.run(*want[-1], g, bc, 1, "f32"))
        want = np.array(want)
        sim = Simulation(_t(x), g, bc, tuned=False)
        sim.set_kernel(2, K, cpl, 0)
        every = torch.zeros((T, 2, R, C), device="cuda")
        sim.step_record(T, every)
        assert np.array_equal(every.cpu().numpy(), want[:T]), (R, C)
        assert np.array_equal(np.array(sim.read_host()), want[T]), (R, C)
        sim.close()
        sim = Simulation(_t(x), g, bc, tuned=False)
        sim.set_kernel(2, K, cpl, 0)
        even = torch.zeros(((T + 1) // 2, 2, R, C), device="cuda")
        sim.step_record_even(T, even)
        assert np.array_equal(even.cpu().numpy(), want[:T:2]), (R, C)
        assert np.array_equal(np.array(sim.read_host()), want[T]), (R, C)
        sim.close()


@pytest.mark.parametrize("bc", ["periodic", "zeroflux"])
@pytest.mark.parametrize("cpl,K", [(1, 8), (2, 12), (4, 8)])
def test_batched_strips_bitwise(cpl, K, bc):
    from paper_2102_10340_amd import Batch
    g, T = W.PLAIN_GENE, 2 * K + 3
    xs = [W.uniform_x(R, C, R + 3 * C) for R, C in _shapes(cpl, K) + [(150, 300)]]
    b = Batch([_t(x) for x in xs], [g] * len(xs), bc)
    b.set_kernel(K, cpl, 11)
    print(f"case batched strips {bc} cpl={cpl} K={K}", flush=True)
    b.step(T)
    for i, x in enumerate(xs):
        got = b.state(i).cpu().numpy()
        u, v = oracle.run(*oracle.init_state(x, 1.0), g, bc, T, "f32")
        assert np.array_equal(got[0], u) and np.array_equal(got[1], v), x.shape
    b.close()


@pytest.mark.parametrize("bc", ["periodic", "zeroflux"])
@pytest.mark.parametrize("cpl", [1, 2, 4])
def test_gray_scott_strips_bitwise(cpl, bc):
    from paper_2102_10340_amd import Simulation
    gs = dict(dt=0.5, F=0.037, k=0.06, Du=0.2, Dv=0.1)
    for R, C in _shapes(cpl, 8):
        print(f"case gray-scott strips {R}x{C} {bc} cpl={cpl}", flush=True)
        rng = np.random.default_rng(R + C)
        u = np.ones((R, C), np.float32)
        v = rng.uniform(0, 0.3, (R, C)).astype(np.float32)
        sim = Simulation.gray_scott(_t(u), _t(v), bc=bc, **gs)
        sim.set_kernel(2, 8, cpl, 9)
        sim.step(19)
        u, v = oracle.gs_run(u, v, gs, bc, 19)
        got = sim.read_host()
        assert np.array_equal(got[0], u) and np.array_equal(got[1], v), (R, C)
        sim.close()


@pytest.mark.parametrize("shape,bc", [((2200, 2200), "periodic"), ((1500, 4004), "zeroflux"),
                                      ((15700, 384), "zeroflux")])
def test_pairs_are_the_larger_grids_choice(shape, bc):
    """Grids beyond the resident tiles' take pairs, whose passes of eight steps and
    the shorter last one match the one-thread-per-cell kernel's bits."""
    from paper_2102_10340_amd import Simulation
    x = _t(W.uniform_x(*shape, 9))
    print(f"case pairs {shape} {bc}", flush=True)
    got, want = (Simulation(x, W.PLAIN_GENE, bc, tuned=False) for _ in range(2))
    cfg = got.pass_config()
    assert (cfg["kind"], cfg["depth"], cfg["cols_per_lane"]) == (2, 8, 4)
    want.set_kernel(1)
    got.step(19)
    want.step(19)
    assert torch.equal(got.state(), want.state())
    got.close()
    want.close()

"""GPU tests of large grids narrow one way: the strips' width follows the columns
(one per lane where two would leave most of a strip idle), and every width gives
the one-thread-per-cell kernel's bits."""
import pytest
import torch

import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("bc", ["zeroflux", "periodic"])
@pytest.mark.parametrize("shape,cols", [((300000, 21), 1), ((200000, 40), 1), ((90000, 96), 2),
                                        ((60000, 128), 1), ((31000, 200), 2)],
                         ids=lambda v: "%dx%d" % v if isinstance(v, tuple) else str(v))
def test_strips_follow_the_width(shape, cols, bc):
    from paper_2102_10340_amd import Simulation
    gen = torch.Generator(device="cuda").manual_seed(cols)
    x = torch.rand(shape, generator=gen, device="cuda") * 2 - 1
    got, want = (Simulation(x, W.PLAIN_GENE, bc, tuned=False) for _ in range(2))
    cfg = got.pass_config()
    assert (cfg["kind"], cfg["depth"], cfg["cols_per_lane"]) == (2, 8, cols), cfg
    want.set_kernel(1)
    print(f"case narrow {shape} {bc}", flush=True)
    for T in (8, 7):
        got.step(T)
        want.step(T)
        assert torch.equal(got.state(), want.state()), T
    got.close()
    want.close()

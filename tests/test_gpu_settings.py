"""GPU tests of pass settings handed back to the library: a value of 0 or a shape
the library itself reported stands for the automatic choice."""
import numpy as np
import torch

import pytest
import workloads as W

pytestmark = pytest.mark.gpu


def test_batch_adjoint_default_rows():
    """Rows of 0 are the automatic ones, with or without the other defaults named,
    and undo a forced cut (the sums of another cut are grouped otherwise)."""
    from paper_2102_10340_amd import Batch
    shapes, S = [(300, 200), (64, 64), (257, 301)], 8
    xs = [torch.from_numpy(W.uniform_x(R, C, R + C)).cuda() for R, C in shapes]
    b = Batch(xs, [W.PLAIN_GENE] * len(xs), "zeroflux", tuned=False)
    states = torch.zeros((S // 2, b.total), device="cuda")
    b.step_record_even(S, states)
    adj0 = torch.rand(b.total, device="cuda") - 0.5

    def dtheta():
        adj, d = adj0.clone(), torch.zeros((len(xs), 8), dtype=torch.float64, device="cuda")
        b.adjoint_even(states, S, adj, torch.empty_like(adj), 0xFF, d)
        return d.cpu().numpy()

    want = dtheta()
    b.set_adjoint_kernel(8, 1, 0)
    assert np.array_equal(dtheta(), want)
    b.set_adjoint_kernel(8, 1, 128)
    assert not np.array_equal(dtheta(), want)
    b.set_adjoint_kernel()
    assert np.array_equal(dtheta(), want)
    b.close()


@pytest.mark.parametrize("shape", [(128, 128), (777, 1301), (2500, 2500), (3000, 100)],
                         ids=lambda s: "%dx%d" % s)
def test_reported_pass_shape_can_be_set(shape):
    """set_kernel takes what pass_config reports, on this grid and on another, and
    steps go on as before."""
    from paper_2102_10340_amd import Simulation
    from paper_2102_10340_amd._lib import RDCNNError
    x = torch.from_numpy(W.uniform_x(*shape, 3)).cuda()
    a, b, other = (Simulation(t, W.PLAIN_GENE, tuned=False) for t in (x, x, x[:64, :64].contiguous()))
    cfg = a.pass_config()
    a.set_kernel(**cfg)
    assert a.pass_config() == cfg
    other.set_kernel(**cfg)
    other.step(9)
    for T in (3, 17):
        assert torch.equal(a.step(T).state(), b.step(T).state())
    for bad in ((4, 0, 4, 8), (4, 17, 4, 8), (4, 8, 1, 8), (4, 8, 4, 0), (5, 8, 4, 8)):
        with pytest.raises(RDCNNError):
            a.set_kernel(*bad)
    for s in (a, b, other):
        s.close()

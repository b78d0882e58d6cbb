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

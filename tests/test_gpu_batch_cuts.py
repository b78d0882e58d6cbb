"""GPU tests of the automatic cuts of a batch into tiles: one small instance, a
few, sizes of one row and one column, a batch either side of the line where tall
tiles take over, plain steps and both recordings in turn on one batch, each bit
for bit equal to the same instance alone on the one-thread-per-cell kernel, and
the reverse pass's (lam, mu) to the one of a forced shape."""
import pytest
import torch

import workloads as W

pytestmark = pytest.mark.gpu

BATCHES = {"one": [(200, 300)], "thin": [(1, 700), (700, 1), (130, 130)],
           "few": [(160, 160), (320, 320), (257, 301)], "below": [(1024, 1024)] * 15,
           "above": [(1024, 1024)] * 20}


@pytest.mark.parametrize("bc", ["periodic", "zeroflux"])
@pytest.mark.parametrize("name", list(BATCHES))
def test_automatic_cuts_bitwise(name, bc):
    from paper_2102_10340_amd import Batch, Simulation
    shapes, T = BATCHES[name], 11
    xs = [torch.from_numpy(W.uniform_x(R, C, R + C)).cuda() for R, C in shapes]
    b = Batch(xs, [W.PLAIN_GENE] * len(xs), bc, tuned=False)
    b.use_lds(False)
    print(f"case batch cuts {name} {bc}", flush=True)
    full = torch.zeros((T, b.total), device="cuda")
    even = torch.zeros(((T + 1) // 2, b.total), device="cuda")
    b.step(T).step_record(T, full).step_record_even(T, even).step_record(T, full)
    for i in {0, len(xs) - 1}:
        ref = Simulation(xs[i], W.PLAIN_GENE, bc, tuned=False)
        ref.set_kernel(1)
        ref.step(2 * T)
        assert torch.equal(b.view(even[0], i), ref.state()), (name, i)
        ref.step(T)
        assert torch.equal(b.view(full[0], i), ref.state()), (name, i)
        ref.step(T)
        assert torch.equal(b.state(i), ref.state()), (name, i)
        ref.close()
    S, outs = 8, []
    adj0 = torch.rand(b.total, device="cuda")
    for forced in (False, True):
        if forced:
            b.set_adjoint_kernel(8, 1, 5)
        adj, tmp = adj0.clone(), torch.empty_like(adj0)
        dtheta = torch.zeros((len(xs), 8), dtype=torch.float64, device="cuda")
        b.adjoint(full, S, adj, tmp, 0xFF, dtheta)
        assert torch.isfinite(dtheta).all()
        outs.append(adj)
    for i in range(len(xs)):  # (the packed layout pads between instances)
        assert torch.equal(b.view(outs[0], i), b.view(outs[1], i)), (name, i)
    b.close()

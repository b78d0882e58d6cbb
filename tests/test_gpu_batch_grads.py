"""GPU tests of a batch's parameter gradients: the automatic cut into tiles and
forced ones give the same dJ/dp of every instance (regrouped float32 sums: within
1e-4 of the instance's largest gradient, the bar two tilings are held to), each with
a gene of its own so that a tile folded into another instance's sums would show, from
one tile an instance to thousands."""
import numpy as np
import pytest
import torch

import workloads as W

pytestmark = pytest.mark.gpu

BATCHES = {"one": [(1024, 1024)], "small": [(16, 20)] * 70, "thin": [(1, 700), (700, 1), (130, 130)],
           "mixed": [(300, 200), (64, 64), (257, 301), (900, 700), (5, 5)],
           "above": [(1024, 1024)] * 20}


@pytest.mark.parametrize("even", [False, True])
@pytest.mark.parametrize("bc", ["periodic", "zeroflux"])
@pytest.mark.parametrize("name", list(BATCHES))
def test_gradients_of_automatic_and_forced_cuts(name, bc, even):
    from paper_2102_10340_amd import Batch
    shapes, S = BATCHES[name], 8
    rng = np.random.default_rng(len(shapes))
    genes = [W.gene(Du=float(rng.uniform(0.02, 0.2)), Dv=float(rng.uniform(0.2, 1.0)),
                    eps=-float(rng.uniform(0.02, 0.2))) for _ in shapes]
    xs = [torch.from_numpy(W.uniform_x(R, C, R + C)).cuda() for R, C in shapes]
    b = Batch(xs, genes, bc, tuned=False)
    states = torch.zeros((S // 2 if even else S, b.total), device="cuda")
    (b.step_record_even if even else b.step_record)(S, states)
    gen = torch.Generator(device="cuda").manual_seed(S)
    adj0 = torch.rand(b.total, generator=gen, device="cuda") * 2 - 1
    got = []
    for forced in (None, (8, 1, 128), (8, 1, 5), (4, 2, 16)):
        print(f"case batch gradients {name} {bc} even={even} cut {forced}", flush=True)
        if forced:
            b.set_adjoint_kernel(*forced)
        adj, tmp = adj0.clone(), torch.empty_like(adj0)
        dtheta = torch.zeros((len(xs), 8), dtype=torch.float64, device="cuda")
        (b.adjoint_even if even else b.adjoint)(states, S, adj, tmp, 0xFF, dtheta)
        got.append(dtheta.cpu().numpy())
    b.close()
    bar = 1e-4 * np.abs(got[1]).max(axis=1, keepdims=True)
    for d in got:
        assert np.all(np.isfinite(d)) and np.all(np.abs(d - got[1]) <= bar)

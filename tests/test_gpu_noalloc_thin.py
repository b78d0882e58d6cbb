"""GPU test of rdcnn_step_bwd_noalloc on grids a few cells thin, where resident
tiles would need more partial-sum slots than its static workspace holds: the call
is accepted with automatic settings and gives rdcnn_step_bwd's bits, whose (lam, mu)
are those of the streamed pairs."""
import pytest
import torch

import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("S", [3, 8])
@pytest.mark.parametrize("bc", ["zeroflux", "periodic"])
@pytest.mark.parametrize("shape", [(2, 1000000), (500000, 1), (400000, 5)], ids=lambda s: "%dx%d" % s)
def test_thin_grids_are_accepted(shape, bc, S):
    from paper_2102_10340_amd import Simulation
    from paper_2102_10340_amd._lib import check, lib
    R, C = shape
    gen = torch.Generator(device="cuda").manual_seed(S)
    x, lam0, mu0 = (torch.rand((R, C), generator=gen, device="cuda") * 2 - 1 for _ in range(3))
    out = []
    for name, forced in (("rdcnn_step_bwd_noalloc", None), ("rdcnn_step_bwd", None),
                         ("rdcnn_step_bwd", (6, 1, 0))):
        print(f"case {name} {R}x{C} S={S} {bc} {forced}", flush=True)
        sim = Simulation(x, W.gene(Du=0.1, Dv=0.5), bc, tuned=False)
        if forced:
            sim.set_adjoint_kernel(*forced)
        st = torch.empty((S + 1, 2, R, C), device="cuda")
        sim.step_record_sparse(S, st)
        lam, mu = lam0.clone(), mu0.clone()
        dth = torch.zeros(8, dtype=torch.float64, device="cuda")
        check(getattr(lib, name)(sim._h, st.data_ptr(), S, lam.data_ptr(), mu.data_ptr(),
                                 dth.data_ptr()))
        torch.cuda.synchronize()
        sim.close()
        out.append((lam, mu, dth))
    for a, b in zip(out[0], out[1]):
        assert torch.equal(a, b)
    assert torch.equal(out[0][0], out[2][0]) and torch.equal(out[0][1], out[2][1])

"""GPU tests of the recording and reverse passes on resident tiles (the automatic
choice up to about six and two million cells): the recorded even states and the
final state are bit for bit those of the streamed recording, and dJ/ds bit for
bit that of the streamed paired passes, over sizes around the tiles' edges and
odd, even, short and long step counts; dJ/dp within 1e-4 of the largest gradient
of the streamed passes' (regrouped float32 sums, the bar two tilings are held
to) and, with non-finite values outside a tile's valid part excluded, never NaN."""
import numpy as np
import pytest
import torch

import workloads as W

pytestmark = pytest.mark.gpu

SHAPES = [(1, 1), (2, 3), (5, 130), (131, 2), (64, 64), (96, 34), (129, 257), (300, 602), (511, 514),
          (1000, 1030), (1400, 1500)]


def _run(x, g, bc, S, kernel, adj_kernel, lam0, mu0):
    from paper_2102_10340_amd import Simulation
    R, C = x.shape
    sim = Simulation(x, g, bc, tuned=False)
    if kernel:
        sim.set_kernel(*kernel)
    if adj_kernel:
        sim.set_adjoint_kernel(*adj_kernel)
    st = torch.full((S + 1, 2, R, C), 7.0, device="cuda")
    sim.step_record_sparse(S, st)
    end = sim.state().clone()
    rec = st.clone()
    lam, mu = lam0.clone(), mu0.clone()
    dth = torch.zeros(8, dtype=torch.float64, device="cuda")
    sim.step_bwd(st, S, lam, mu, dth)
    sim.close()
    return rec, end, lam, mu, dth.cpu().numpy()


@pytest.mark.parametrize("S", [1, 2, 3, 10, 27])
@pytest.mark.parametrize("bc", ["periodic", "zeroflux"])
@pytest.mark.parametrize("shape", SHAPES, ids=lambda s: "%dx%d" % s)
def test_tile_record_and_adjoint_match_streamed(shape, bc, S):
    R, C = shape
    g = W.gene(W.PAPER_DEFAULT_GENE, k3=0.45, Du=0.08, Dv=0.6) if bc == "periodic" else \
        W.gene(Du=0.1, Dv=0.5)
    x = torch.from_numpy(W.uniform_x(R, C, R + C)).cuda()
    gen = torch.Generator(device="cuda").manual_seed(S)
    lam0 = torch.randn((R, C), generator=gen, device="cuda")
    mu0 = torch.randn((R, C), generator=gen, device="cuda")
    print(f"case tile record/adjoint {shape} {bc} S={S}", flush=True)
    a = _run(x, g, bc, S, None, None, lam0, mu0)
    b = _run(x, g, bc, S, (2, 8, 1, 0), (6, 1, 0), lam0, mu0)
    for what, p, q in zip(("recorded states", "final state", "lam", "mu"), a, b):
        assert torch.equal(p, q), what
    assert np.all(np.isfinite(a[4]))
    assert np.all(np.abs(a[4] - b[4]) <= 1e-4 * np.abs(b[4]).max()), (a[4], b[4])


def test_tile_adjoint_grad_mask():
    """Without the three lam-weighted sums the other gradients keep their bits."""
    from paper_2102_10340_amd import Simulation
    R, C, S = 200, 260, 14
    x = torch.from_numpy(W.uniform_x(R, C, 1)).cuda()
    out = []
    for mask in (0xFF, 0xCE):
        sim = Simulation(x, W.PLAIN_GENE, "zeroflux", tuned=False)
        sim.set_grad_mask(mask)
        st = torch.empty((S + 1, 2, R, C), device="cuda")
        sim.step_record_sparse(S, st)
        lam, mu = x.clone(), torch.zeros_like(x)
        dth = torch.zeros(8, dtype=torch.float64, device="cuda")
        sim.step_bwd(st, S, lam, mu, dth)
        out.append((lam, dth.cpu().numpy()))
        sim.close()
    assert torch.equal(out[0][0], out[1][0])
    for q in range(8):
        if 0xCE >> q & 1:
            assert out[0][1][q] == out[1][1][q], q
        else:
            assert np.isnan(out[1][1][q]), q

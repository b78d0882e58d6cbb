"""GPU tests of device reads into memory that the one-launch read may not take: it
is left to copies, whose results and refusals such reads had."""
import ctypes

import pytest
import torch

import workloads as W

pytestmark = pytest.mark.gpu

R, C = 40, 50


def _sim():
    from paper_2102_10340_amd import Simulation
    sim = Simulation(torch.from_numpy(W.uniform_x(R, C, 3)).cuda(), W.PLAIN_GENE, tuned=False)
    sim.step(5)
    return sim


def _may(sim, u, v):
    from paper_2102_10340_amd import _lib
    f = _lib.lib._ZN2rd15kernel_may_readEPKfxS1_S1_
    f.argtypes = [ctypes.c_void_p, ctypes.c_longlong, ctypes.c_void_p, ctypes.c_void_p]
    f.restype = ctypes.c_bool
    return f(sim.state().data_ptr(), R * C, u, v)


def test_what_the_kernel_may_read():
    hip = ctypes.CDLL("libamdhip64.so")
    sim = _sim()
    n = R * C
    ok = torch.empty(4 * n, device="cuda")
    u, v = ok.data_ptr(), ok.data_ptr() + 8 * n
    assert _may(sim, u, v)
    assert _may(sim, u, u + 4 * n)  # side by side
    assert not _may(sim, u, u)  # one over the other
    assert not _may(sim, u, u + 4 * n - 4)
    assert not _may(sim, u + 2, v)  # between floats
    state = sim.state().data_ptr()
    assert not _may(sim, state + 4 * n, v)  # over the state
    assert not _may(sim, u, state - 4 * n + 4)
    host = torch.empty(n)
    assert not _may(sim, host.data_ptr(), v)
    assert not _may(sim, u, torch.empty(n, pin_memory=True).data_ptr())
    small = ctypes.c_void_p()  # an allocation shorter than a plane
    assert hip.hipMalloc(ctypes.byref(small), ctypes.c_size_t(4 * n - 64)) == 0
    assert not _may(sim, small.value, v)
    assert not _may(sim, u, small.value)
    assert hip.hipFree(small) == 0
    sim.close()


def test_reads_over_the_state_and_each_other_are_as_two_copies():
    """The second plane is read after the first has been written."""
    from paper_2102_10340_amd._lib import check, lib
    n = R * C
    sim = _sim()
    st = sim.state()
    want_u, want_v = st[0].clone(), st[1].clone()
    out = torch.empty(n, device="cuda")
    check(lib.rdcnn_read(sim._h, st[1].data_ptr(), out.data_ptr(), 0))
    assert torch.equal(st[1], want_u) and torch.equal(out.view(R, C), want_u)
    sim.write_state(want_u, want_v)
    pair = torch.empty(n + 8, device="cuda")
    check(lib.rdcnn_read(sim._h, pair.data_ptr() + 32, pair.data_ptr(), 0))
    assert torch.equal(pair[:n].view(R, C), want_v)
    assert torch.equal(pair[n:], want_u.reshape(-1)[-8:])
    bytes_ = torch.zeros(8 * n + 8, dtype=torch.uint8, device="cuda")  # not on a float's address
    check(lib.rdcnn_read(sim._h, bytes_.data_ptr() + 2, bytes_.data_ptr() + 4 * n + 2, 0))
    got = bytes_[2:8 * n + 2].clone().view(torch.float32)
    assert torch.equal(got[:n].view(R, C), want_u) and torch.equal(got[n:].view(R, C), want_v)
    sim.close()


@pytest.mark.parametrize("shape", [(1, 1), (3, 5), (64, 64), (513, 1023), (1025, 2048), (1449, 1449)])
@pytest.mark.parametrize("offset", [0, 1])  # offset in floats from a vector's address
def test_one_launch_reads_every_size(shape, offset):
    """One cell to several trips of the kernel's grid, vectors and single floats."""
    from paper_2102_10340_amd import Simulation
    from paper_2102_10340_amd._lib import check, lib
    n = shape[0] * shape[1]
    sim = Simulation(torch.from_numpy(W.uniform_x(*shape, 3)).cuda(), W.PLAIN_GENE, tuned=False)
    sim.step(1)
    out = torch.full((2 * n + offset + 4,), -7.0, device="cuda")
    u = out.data_ptr() + 4 * offset
    check(lib.rdcnn_read(sim._h, u, u + 4 * n, 0))
    st = sim.state()
    assert torch.equal(out[offset:offset + n].view(shape), st[0])
    assert torch.equal(out[offset + n:offset + 2 * n].view(shape), st[1])
    assert bool((out[:offset] == -7).all()) and bool((out[offset + 2 * n:] == -7).all())
    sim.close()

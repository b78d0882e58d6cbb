"""GPU tests of steps, recordings and reads captured into a caller's
graph: replays, with eager work between them, give the eager results.  The sizes take
resident tiles with little and with more than 64 KB of LDS, streamed passes, one-launch
reads and copied ones."""
import pytest
import torch

import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shape,T", [((128, 128), 10), ((1536, 1536), 20), ((1024, 1024), 3),
                                     ((2000, 90), 12)], ids=lambda v: str(v))
def test_captured_steps_and_reads(shape, T):
    from paper_2102_10340_amd import Simulation
    x = torch.from_numpy(W.uniform_x(*shape, 3)).cuda()
    s = torch.cuda.Stream()
    s.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(s):
        a, b = (Simulation(x, W.PLAIN_GENE, tuned=False) for _ in range(2))
        u, v = torch.zeros_like(x), torch.zeros_like(x)
        st = torch.empty((T + 1, 2, *shape), device="cuda")
        for sim in (a, b):  # first uses
            sim.step(2 * T)
            sim.step_record_sparse(T, st)
            sim.step_record_sparse(T, st)
        s.synchronize()
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g, stream=s):
            a.step(T).step(T)  # an even number of runs: the state ends where it began
            a.step_record_sparse(T, st).step_record_sparse(T, st)
            a.read_into(u, v)
        for k in range(3):
            print(f"case capture {shape} T={T} replay {k}", flush=True)
            g.replay()
            s.synchronize()
            b.step(T).step(T)
            rec = torch.empty_like(st)
            b.step_record_sparse(T, rec).step_record_sparse(T, rec)
            want = b.read()
            assert torch.equal(u, want[0]) and torch.equal(v, want[1]), k
            assert torch.equal(st[0:T:2], rec[0:T:2]), k
        a.close()
        b.close()

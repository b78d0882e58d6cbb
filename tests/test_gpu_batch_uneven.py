"""GPU tests of batches of very uneven sizes: creation starts every instance from
its own image, however large the largest one is."""
import pytest
import torch

import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("big,small,n", [((4096, 4096), (8, 8), 8300), ((300, 500), (1, 1), 3),
                                         ((64, 128), (91, 90), 40)],
                         ids=lambda v: "%dx%d" % v if isinstance(v, tuple) else str(v))
def test_uneven_batch_starts_from_its_images(big, small, n):
    from paper_2102_10340_amd import Batch
    gen = torch.Generator(device="cuda").manual_seed(n)
    shapes = [small] * (n // 2) + [big] + [small] * (n - n // 2)
    xs = [torch.rand(s, generator=gen, device="cuda") for s in shapes]
    print(f"case uneven batch {big} among {n} of {small}", flush=True)
    b = Batch(xs, [W.PLAIN_GENE] * len(xs), "zeroflux", ka=0.5, tuned=False)
    for i in {0, 1, n // 2 - 1, n // 2, n // 2 + 1, n}:
        st = b.state(i)
        assert torch.equal(st[0], 0.5 * xs[i]) and torch.equal(st[1], st[0]), i
    b.close()

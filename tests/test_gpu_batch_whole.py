"""GPU tests of the batch instances held whole in one workgroup's registers:
bit for bit equal to the float32 oracle for every number of rows per block
(1 to 6), both column widths, grids that fill the 32 lanes and grids that wrap
inside them, one block and many, odd and even step counts, both rules, and
mixed with instances the other kernels take."""
import numpy as np
import pytest
import torch

import oracle
import workloads as W

pytestmark = pytest.mark.gpu

# rows per block 4, 4, 4, 4, 3, 5, 2, 6, 5, 1, 4, 6, 3; (129, 200) is streamed,
# (17, 33) has an odd width and stays in LDS
SHAPES = [(128, 128), (64, 64), (100, 100), (12, 2), (96, 68), (25, 40), (2, 128), (186, 64),
          (160, 32), (31, 126), (31, 64), (4, 128), (126, 120), (93, 128), (129, 200), (17, 33)]


@pytest.mark.parametrize("T", [1, 2, 23, 40])
@pytest.mark.parametrize("bc", ["zeroflux", "periodic"])
def test_whole_instances_bitwise(bc, T):
    from paper_2102_10340_amd import Batch
    rng = np.random.default_rng(T)
    xs = [W.uniform_x(R, C, 5 * R + C) for R, C in SHAPES]
    base = W.PAPER_DEFAULT_GENE if bc == "periodic" else W.PLAIN_GENE
    genes = [W.gene(base, Du=rng.uniform(0.01, 0.2)) for _ in xs]
    b = Batch([torch.from_numpy(x).cuda() for x in xs], genes, bc)
    print(f"case whole instances {bc} T={T}: {b.lds_instances()} held whole", flush=True)
    assert b.lds_instances() >= len(SHAPES) - 2
    b.step(T).step(T)
    for i, (x, g) in enumerate(zip(xs, genes)):
        got = b.state(i).cpu().numpy()
        ou, ov = oracle.run(*oracle.init_state(x, 1.0), g, bc, 2 * T, "f32")
        assert np.array_equal(got[0], ou) and np.array_equal(got[1], ov), x.shape
    b.close()

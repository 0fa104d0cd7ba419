"""Order of a sphere's link sums on the GPU (Eqs. netforce, torque).

The links of a sphere are summed within waves in a fixed order; only what the waves add to
the sphere's accumulators (copies, by block) comes in any order, and two additions to a
cleared accumulator commute.  Spheres of one node whose links fill three rows of one chunk of
planes, two in one tile of four rows and one in the next, add at most twice to each copy, so
two runs give the same bits.  A sum over a block that its lanes add to as they come does not.
"""
import numpy as np
import pytest

import paper_1712_07028_amd as fsl
from paper_1712_07028_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _built():
    import torch

    if not torch.cuda.is_available():
        pytest.skip("no HIP device")
    fsl.load_library()


@pytest.mark.parametrize("storage", [0, 1, 2])
def test_link_sums_repeat_to_the_bit(storage):
    rng = np.random.Generator(np.random.PCG64(3))
    # 4 x 16 tile columns of 33 chunks of four planes: neighbouring columns add to different copies
    n = (256, 64, 132)
    j, i, k = np.meshgrid(np.arange(8), np.arange(12), np.arange(8), indexing="ij")
    x = np.stack([10 + 20 * i, 8 * j + 3, 16 * k + 9], axis=-1).reshape(-1, 3) + rng.uniform(-0.15, 0.15, (768, 3))
    p = W.Particles(x=x, u=rng.uniform(-0.002, 0.002, x.shape), omega=rng.uniform(-0.004, 0.004, x.shape),
                    R=np.full(len(x), 0.7), rho_p=np.full(len(x), 2.5))
    w = W.Workload(name="dots", n=n, trt=True, tau=0.55, g=(0.0, 0.0, -1e-6), zs=-1.0, steps=0, periodic=(0, 0, 0),
                   particles=p, storage=storage)
    runs = []
    for _ in range(2):
        s = fsl.Sim(w)
        for _ in range(5):
            s.step(10)
            runs.append(s.particles_get())
        s.close()
    for a, b in zip(runs[:5], runs[5:]):
        assert np.abs(a["x"] - x).max() < 0.3 and np.abs(a["F"]).max() > 0.0
        for key in ("x", "u", "omega", "F", "T"):
            np.testing.assert_array_equal(a[key], b[key], err_msg=key)

"""Single steps of a small sphere table on boxes at either side of the axis length up to which
every pair is tested (in FP32 first); longer boxes take the grid of pairs and a launch per
phase.  Pairs with acting lubrication near the far end, against the oracle."""
import numpy as np
import pytest

import oracle as O
import paper_1712_07028_amd as fsl
from paper_1712_07028_amd import workloads as W

from gpu_common import compare_step, transfer

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _built():
    O.build(force=False)
    import torch

    if not torch.cuda.is_available():
        pytest.skip("no HIP device")
    fsl.load_library()


@pytest.mark.parametrize("nx,per", [(65536, 0), (65544, 0), (65544, 1)])
def test_single_step_on_a_long_box(nx, per):
    """Bars of the single-step cases."""
    rng = np.random.Generator(np.random.PCG64(5))
    R = 1.6
    x = np.array([[nx - 40.0 + (2 * R + 0.45) * i, 5.0 + (2 * R + 0.4) * j, 5.0] for i in range(9) for j in range(2)])
    x += rng.uniform(-0.05, 0.05, size=x.shape)
    u = rng.normal(size=x.shape)
    u *= 0.02 / np.linalg.norm(u, axis=1)[:, None]
    p = W.Particles(x=x, u=u, omega=rng.uniform(-0.004, 0.004, size=x.shape), R=np.full(len(x), R),
                    rho_p=np.full(len(x), 2.5))
    w = W.Workload(name="long", n=(nx, 14, 10), trt=True, tau=0.6, g=(0, 0, -1e-5), zs=-1.0, steps=0,
                   periodic=(per, 0, 0), particles=p)
    o, s = O.Oracle(w), fsl.Sim(w)
    transfer(o, s, w)
    o.step(1)
    s.step(1)
    s.sync()
    print(nx, per, compare_step(o, s, w), flush=True)
    s.close()
    o.close()

"""Per-phase timing: every phase of a step is counted once a step, whatever launches it takes on the
box and the table at hand (the curvature only with surface tension, the spheres' phases only with
spheres)."""
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


@pytest.mark.parametrize("count,gas,sigma", [(0, True, 0.0), (0, False, 0.0), (0, False, 0.004), (12, True, 0.004), (12, False, 0.0),
                                             (2060, True, 0.0)])
def test_phases_count_once_a_step(count, gas, sigma):
    k, j, i = np.meshgrid(np.arange(13), np.arange(13), np.arange(13), indexing="ij")
    x = (3.0 + 4.0 * np.stack([i, j, k], axis=-1).reshape(-1, 3))[:count]
    p = W.Particles(x=x, u=np.zeros_like(x), omega=np.zeros_like(x), R=np.full(count, 1.2), rho_p=np.full(count, 2.5))
    w = W.Workload(name="phases", n=(56, 56, 64), trt=True, tau=0.6, g=(0, 0, -1e-5), zs=58.0 if gas else -1.0,
                   steps=0, sigma=sigma, particles=p if count else None)
    s = fsl.Sim(w)
    s.step(2)
    s.profile(True)
    s.profile_get()
    s.step(7)
    n = {name: v[1] for name, v in s.profile_get().items()}
    spheres = 7 if count else 0
    assert n == {"stream_collide": 7, "conversions": 7, "bubbles": 7, "particle_forces": spheres,
                 "particle_substeps": spheres, "coverage": spheres, "curvature": 7 if sigma else 0, "split": 7}
    s.close()

"""Single steps of sphere tables at the sizes where the particle update changes its form
(lone spheres in blocks of 64, one block of 1,024 threads for those with a listed pair, the
grid of pairs and a launch per half substep beyond 2,048), with the launches of a step joined
and apart (per-phase timing), against the oracle."""
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


def packed(count, gap, gas):
    """count spheres of radius 1.6 at the sites of a grid (surface gaps around `gap`), every
    one moving at 0.02 in a direction of its own."""
    R, rng = 1.6, np.random.Generator(np.random.PCG64(count))
    a = 2 * R + gap
    k = 13
    i = np.arange(count)
    x = 3.0 + a * np.stack([i % k, i // k % k, i // (k * k)], axis=1)
    x += rng.uniform(-1, 1, size=x.shape) * min(0.15, gap / 4.5)
    u = rng.normal(size=x.shape)
    u *= 0.02 / np.linalg.norm(u, axis=1)[:, None]
    p = W.Particles(x=x, u=u, omega=rng.uniform(-0.004, 0.004, size=x.shape), R=np.full(count, R),
                    rho_p=np.full(count, 2.5))
    nz = 72 if gas else 70
    return W.Workload(name="packed", n=(68, 67, nz + 8 if gas else nz), trt=True, tau=0.6, g=(0, 0, -1e-5),
                      zs=float(nz) if gas else -1.0, steps=0, particles=p)


# gaps of 1.8: a few percent of the spheres have a listed pair (reach 5/3); gaps of 0.45: all
# have, about three each, and lubrication acts
@pytest.mark.parametrize("count,gap,gas", [(1, 1.8, True), (64, 1.8, True), (65, 1.8, False), (1024, 1.8, True),
                                           (1025, 1.8, False), (2048, 1.8, True), (2049, 1.8, True), (600, 0.45, True),
                                           (1100, 0.45, False), (2048, 0.45, True)])
def test_single_step_of_tables(count, gap, gas):
    """Bars of the single-step cases."""
    w = packed(count, gap, gas)
    o = O.Oracle(w)
    o.step(2)
    sims = []
    for apart in (False, True):
        s = fsl.Sim(w)
        transfer(o, s, w)
        s.profile(apart)
        sims.append(s)
    # the table handed to both sides restarts the update: the last transfer serves both
    o.step(1)
    for s in sims:
        s.step(1)
        s.sync()
        print(count, gap, gas, compare_step(o, s, w), flush=True)
        s.close()
    o.close()

"""A sphere that leaves the box in a substep and is back by the end of the step is an error on tables
above 512 spheres (whatever takes their substeps), and none on smaller ones.  The sphere moves in
the gas above a pool, where no link acts on it: 35 cells per substep, reversed at either face.
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


@pytest.mark.parametrize("count,paired", [(512, False), (512, True), (513, False), (513, True), (1025, True), (2049, False)])
def test_a_centre_outside_between_two_substeps(count, paired):
    n = (40, 72, 88)
    j, i, k = np.meshgrid(np.arange(17), np.arange(9), np.arange(15), indexing="ij")
    x = np.stack([3.5 + 4 * i, 3.5 + 4 * j, 3.5 + 4 * k], axis=-1).reshape(-1, 3)[:count].astype(float)
    x[-1] = (10.0, 36.0, 78.0)
    u = np.zeros_like(x)
    u[-1, 0] = 350.0
    if paired:  # a second sphere within reach (a listed pair), no nodes next to one another
        x[-2] = (10.0, 39.5, 78.0)
    p = W.Particles(x=x, u=u, omega=np.zeros_like(x), R=np.full(count, 1.0), rho_p=np.full(count, 2.5))
    w = W.Workload(name="out", n=n, trt=True, tau=0.6, g=(0.0, 0.0, 0.0), zs=68.0, steps=0, periodic=(0, 0, 0), particles=p)
    s = fsl.Sim(w)
    s.step(1)
    if count > 512:
        with pytest.raises(fsl.FslError, match="left the box"):
            s.sync()
    else:
        s.sync()
    s.close()

"""The march's three forms of addresses (byte offsets within a pair of planes, element offsets on boxes
beyond that, 64 bits) read and write the same words: single steps of one state with each, on a bed
with walls, spheres and a bubble and on a periodic liquid box, agree to the last bit."""
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


def state(w, form, monkeypatch):
    if form:
        monkeypatch.setenv("FSL_WIDE_OFFSETS", form)
    else:
        monkeypatch.delenv("FSL_WIDE_OFFSETS", raising=False)
    s = fsl.Sim(w)
    s.step(1)
    fl = s.get(fsl.FIELD_FLAGS)
    f = s.get(fsl.FIELD_F)[:, (fl == fsl.LIQ) | (fl == fsl.IFC)]
    s.close()
    return fl, f


@pytest.mark.parametrize("periodic", [0, 1])
@pytest.mark.parametrize("storage", [0, 1, 2])
def test_forms_agree_to_the_bit(storage, periodic, monkeypatch):
    n = (130, 37, 41)
    bub = (65.0, 18.0, 11.0, 6.0, 1.0)
    p = W.particle_bed(40, 3.5, n, 33.0, bub, seed=7, rho_p=2.5, vel_range=0.01)
    w = W.Workload(name="forms", n=n, trt=True, tau=0.55, g=(1e-5, 0, -2e-5), zs=-1.0 if periodic else 33.0, steps=0,
                   periodic=(periodic,) * 3, gas_spheres=[] if periodic else [bub], particles=p, storage=storage)
    fl, f = state(w, "", monkeypatch)
    for form in ("pair", "1"):
        gl, g = state(w, form, monkeypatch)
        np.testing.assert_array_equal(fl, gl)
        np.testing.assert_array_equal(f, g)

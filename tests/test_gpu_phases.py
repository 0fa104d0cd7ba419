"""The conversion phases and the labelling of a split in both of their forms (one launch
with barriers between the phases up to 4 M cells, a launch per phase beyond) against the
oracle: many conversions of every kind at once, and gas that falls apart."""
import sys

import numpy as np
import pytest

import oracle as O
import paper_1712_07028_amd as fsl

from gpu_common import compare_step
from test_gpu_split import compare_bubbles, copy_fields
from test_oracle_split import ball, hand_state

pytestmark = pytest.mark.gpu

SMALL, LARGE = (40, 36, 26), (163, 162, 161)  # 37 thousand and 4.25 M cells


@pytest.fixture(scope="module", autouse=True)
def _built():
    O.build(force=False)
    import torch

    if not torch.cuda.is_available():
        pytest.skip("no HIP device")
    fsl.load_library()


def sim_of(o, st):
    s = fsl.Sim(st["w"])
    copy_fields(o, s)
    for x in (o, s):
        x.bubbles_set([0.0, st["M"]], [0, 1], [0, 1])
    return s


@pytest.mark.parametrize("n,fill", [(SMALL, (0.12, 0.12)), (SMALL, (0.004, 0.0)), (SMALL, (0.0, 0.004)),
                                    (LARGE, (0.12, 0.12))])
def test_many_conversions_at_once(n, fill):
    """A slab of gas whose interface cells fill, empty or stay at random (some 500 cells,
    or a handful; the gas stays in fewer than the 64 parts of the table): conflict rule, closure, excess mass and merges after one and two steps.
    Bars of the single-step cases."""
    print("conversions", n, fill, flush=True)
    gas = np.zeros((n[2], n[1], n[0]), bool)
    gas[9:13, 3:33, 4:36] = True
    o, st = hand_state(n, gas)
    rng = np.random.Generator(np.random.PCG64(11))
    k = int(st["ifc"].sum())
    r = rng.random(k)
    phi = np.where(r < fill[0], 1.002, np.where(r < fill[0] + fill[1], -0.002, 0.5))
    o.close()
    o, st = hand_state(n, gas, phi_ifc=phi)
    s = sim_of(o, st)
    for _ in range(2):
        o.step(1)
        s.step(1)
        s.sync()
        print(compare_step(o, s, st["w"]), flush=True)
        sys.stdout.flush()
    o.close()
    s.close()


@pytest.mark.parametrize("n", [SMALL, LARGE])
def test_split_labelling(n):
    """Three blobs set as one bubble: labelled, numbered and given their gas masses as the
    oracle does (bars of the splitting tests)."""
    gas = ball(n, (8.3, 9.0, 8.0), 3.6) | ball(n, (24.0, 20.5, 12.0), 5.4) | ball(n, (9.0, 27.0, 17.0), 2.2)
    o, st = hand_state(n, gas, rho_g=1.01)
    s = sim_of(o, st)
    assert compare_bubbles(o, s) == 4
    o.close()
    s.close()

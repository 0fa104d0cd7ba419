"""Phases of a step that share launches: the labelling of a step in one launch and in a launch per
phase, cells covered in the step in which their bubble merges, a box that gets gas after steps
without any were captured, and the 16-bit forms of the launches of small sphere tables."""
import numpy as np
import pytest

import oracle as O
import paper_1712_07028_amd as fsl
from paper_1712_07028_amd import workloads as W

from gpu_common import compare_step
from test_gpu_graph import agree
from test_gpu_phases import LARGE, SMALL
from test_gpu_split import compare_bubbles, copy_fields, stepped, twin
from test_gpu_tables import packed
from test_oracle_split import ball, hand_state, interface_of

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _built():
    O.build(force=False)
    import torch

    if not torch.cuda.is_available():
        pytest.skip("no HIP device")
    fsl.load_library()


@pytest.mark.parametrize("n", [SMALL, LARGE])
def test_gas_falls_apart_in_a_step(n):
    """A neck of gas closed by conversions, so that the test of the step asks for the labelling (boxes
    up to 4 M cells take it in one launch): bars of the splitting tests."""
    gas = ball(n, (6.0, 8.0, 9.0), 3.0) | ball(n, (19.0, 8.0, 9.0), 3.0)
    gas[9, 8, 8:19] = True
    z, y, x = np.nonzero(interface_of(gas))
    full = (x >= 11) & (x <= 14) & (abs(y - 8) <= 1) & (abs(z - 9) <= 1)
    o, s, st = twin(n, gas, phi_ifc=np.where(full, 1.001, 0.5))
    assert stepped(o, s, st["w"], 3, "conversions") is not None
    o.close()
    s.close()


def test_cells_covered_as_their_bubble_merges():
    """Bubbles 1 and 2 merge through a layer that empties, while a sphere covers a gas cell of bubble
    2: every gas and interface cell carries the root, two steps on as well."""
    n = (26, 16, 16)
    gas = np.zeros((16, 16, 26), bool)
    gas[3:8, 3:8, 2:6] = True
    gas[3:8, 3:8, 7:11] = True
    z, y, x = np.nonzero(interface_of(gas))
    # the axis node x = 10 lies 3.01 from the centre, 2.99 after the step
    p = W.Particles(x=np.array([[13.01, 5.0, 5.0]]), u=np.array([[-0.02, 0.0, 0.0]]), omega=np.zeros((1, 3)),
                    R=np.array([3.0]), rho_p=np.array([50.0]))
    o, s, st = twin(n, gas, phi_ifc=np.where(x == 6, 0.0, 0.5), particles=p)  # the two parts split
    before = s.get(fsl.FIELD_FLAGS)
    assert before[5, 5, 10] == fsl.GAS and s.get(fsl.FIELD_BUBBLE_ID)[5, 5, 10] == 2
    for _ in range(3):
        o.step(1)
        s.step(1)
        s.sync()
        print(compare_step(o, s, st["w"]), flush=True)
        compare_bubbles(o, s, rtol=1e-6)
        fl, b = s.get(fsl.FIELD_FLAGS), s.get(fsl.FIELD_BUBBLE_ID)
        assert fl[5, 5, 10] == fsl.SOL
        assert set(np.unique(b[(fl == fsl.GAS) | (fl == fsl.IFC)])) == {1}
    o.close()
    s.close()


def test_gas_after_steps_without_any():
    """A liquid box steps from a captured graph, gets a bubble through the field setters, steps on,
    and loses it again: as steps one at a time (bars of the graph tests)."""
    n = (24, 22, 20)
    o, st = hand_state(n, ball(n, (11.0, 10.0, 9.0), 4.0), rho_g=1.01, g=(0, 0, -1e-5))
    g, e = fsl.Sim(st["w"]), fsl.Sim(st["w"])
    liquid = {k: g.get(k) for k in (fsl.FIELD_FLAGS, fsl.FIELD_F, fsl.FIELD_MASS, fsl.FIELD_PHI, fsl.FIELD_BUBBLE_ID)}

    def run():
        for k in (20, 9):
            g.step(k)
            for _ in range(k):
                e.step(1)
        agree(g, e, 1e-12)

    run()
    for s in (g, e):
        copy_fields(o, s)
        s.bubbles_set([0.0, st["M"]], [0, 1], [0, 1])
    run()
    assert alive(g) == [1]
    for s in (g, e):
        for k, v in liquid.items():
            s.set(k, v)
    run()
    assert alive(g) == []
    for s in (o, g, e):
        s.close()


def alive(s):
    return [i for i, b in enumerate(s.bubbles()) if b["alive"]]


@pytest.mark.parametrize("storage", [1, 2])
@pytest.mark.parametrize("count,gap,gas", [(64, 1.8, True), (1025, 1.8, True), (2048, 0.45, False), (2049, 1.8, True)])
def test_sixteen_bit_tables_joined_and_apart(count, gap, gas, storage):
    """Three steps with the launches joined and apart (per-phase timing): cell types, owners and
    populations to the bit, forces to the rounding of their sums."""
    w = packed(count, gap, gas).replace(storage=storage)
    out = []
    for apart in (False, True):
        s = fsl.Sim(w)
        s.profile(apart)
        s.step(3)
        s.sync()
        fl = s.get(fsl.FIELD_FLAGS)
        out.append((fl, s.get(fsl.FIELD_PID), s.get(fsl.FIELD_F)[:, (fl == fsl.LIQ) | (fl == fsl.IFC)],
                    s.particles_get()))
        s.close()
    a, b = out
    for k in range(3):
        np.testing.assert_array_equal(a[k], b[k])
    for k in ("x", "u", "omega", "F", "T"):
        assert np.abs(a[3][k] - b[3][k]).max() <= 1e-9 * max(1.0, np.abs(a[3][k]).max()), k

"""FP64 boxes on either side of the densities at which the SF pass (45 neighbours on
average) and the force and force-adjoint passes (80) go over to the polynomials of
the angular etas: energies, forces and the weight gradient against the oracle at
the FP64 bars, and the same values from a handle that has seen denser boxes."""
import numpy as np
import pytest

from common import oracle_water
from gpu_common import check_fp64, make_potential, run, say, to_dev
from paper_2002_00054_amd import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("mean", [20, 44, 46, 79, 81, 110])
def test_both_sides_of_the_lines(mean):
    import torch

    unit = 3 / synth.WATER_SPACING ** 3 * 4 / 3 * np.pi * 6.0 ** 3
    box = lambda m, seed: synth.water_box(9, seed, spacing=synth.WATER_SPACING * (unit / m) ** (1 / 3))
    b = box(mean, 7)
    say("polynomial rule", mean, b.n_atoms / np.prod(b.box) * 4 / 3 * np.pi * 216)
    ref = oracle_water().compute(b.pos, b.types, b.box, use_cells=True)
    gF = np.random.default_rng(1).standard_normal((b.n_atoms, 3))

    def results(pot):
        e, ei, f = run(pot, b)
        pos, types = to_dev(b, torch.float64)
        g = pot.backward(pos, types, [0, b.n_atoms], [b.box], torch.tensor([0.3], device="cuda"),
                         torch.tensor(gF, device="cuda")).cpu().numpy()
        return ei, f, g

    pot, used = make_potential("fp64"), make_potential("fp64")
    ei, f, g = results(pot)
    check_fp64(ei, f, ref["Ei"], ref["F"])
    run(used, box(130, 8))
    ei2, f2, g2 = results(used)
    assert np.array_equal(ei, ei2)
    assert np.max(np.abs(f - f2)) <= 1e-12 * np.max(np.abs(f)) and np.max(np.abs(g - g2)) <= 1e-12 * np.max(np.abs(g))
    pot.close()
    used.close()

"""Compact neighbour rows longer than the padded capacity that the mean density
suggests (atoms in a fifth of a long box: 48 slots, rows of over 100): the LDS
rows of the pair passes have to follow the rows, not that capacity."""
import numpy as np
import pytest

from common import oracle_water
from gpu_common import check_fp64, make_potential, run, say
from paper_2002_00054_amd import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("side", [5, 9])  # two waves per centre, and one
def test_compact_rows_beyond_the_padded_capacity(side):
    b = synth.water_box(side, 2)
    b = synth.Box(pos=b.pos, types=b.types, box=np.array([b.box[0], b.box[1], 5 * b.box[2]]))
    ref = oracle_water().compute(b.pos, b.types, b.box, use_cells=True)
    pot = make_potential("fp64")
    pot.set_list_layout("compact")
    for call in range(2):
        e, ei, f = run(pot, b)
        say("compact rows", b.n_atoms, "call", call, "capacity", pot.neighbor_capacity)
        assert pot.neighbor_capacity < 100  # the padded capacity did not grow
        check_fp64(ei, f, ref["Ei"], ref["F"])
    pot.close()

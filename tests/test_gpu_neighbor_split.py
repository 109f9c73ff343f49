"""Neighbour builds whose cells share their centres among several workgroups:
one cell per axis up to more cells than workgroups fit on the card, cells with
fewer centres than workgroups (and none), cells of more than 64 centres and of
more candidates than one tile, for one structure, for batches, and for the
index and compact rows. FP64 against the oracle at the FP64 bars; the layouts
among themselves to 1e-12 (the same rows)."""
import numpy as np
import pytest

from common import oracle_water
from gpu_common import check_fp64, make_potential, run, say
from paper_2002_00054_amd import synth

pytestmark = pytest.mark.gpu


def _box(kind):
    if kind == "slab":  # atoms in a fifth of a long box: most cells are empty
        b = synth.water_box(5, 2)
        return synth.Box(pos=b.pos, types=b.types, box=np.array([b.box[0], b.box[1], 5 * b.box[2]]))
    if kind == "droplet":  # the dense half of a wide box: uneven cells
        b = synth.water_box(9, 3)
        keep = np.linalg.norm(b.pos - b.box / 2, axis=1) < 10.0
        return synth.Box(pos=b.pos[keep], types=b.types[keep], box=b.box)
    if kind == "dense":  # about 170 centres in a cell, some 1,300 candidates
        b = synth.water_box(8, 4, spacing=0.62 * synth.WATER_SPACING)
        return b
    if kind == "few":  # fewer atoms than cells
        b = synth.water_box(9, 5)
        return synth.Box(pos=b.pos[::40], types=b.types[::40], box=b.box)
    return synth.water_box(kind, 6)


@pytest.mark.parametrize("kind", [4, 7, 12, 19, "slab", "droplet", "dense", "few"])
def test_shared_cells_match_oracle(kind):
    b = _box(kind)
    say("neighbour split", kind, b.n_atoms)
    ref = oracle_water().compute(b.pos, b.types, b.box, use_cells=True)
    got = {}
    for layout in ("padded", "index", "compact"):
        pot = make_potential("fp64")
        pot.set_list_layout(layout)
        for _ in range(2):  # the second call launches ahead of the build's counts
            e, ei, f = run(pot, b)
            check_fp64(ei, f, ref["Ei"], ref["F"])
        got[layout] = (ei, f)
        pot.close()
    for layout in ("index", "compact"):
        assert np.max(np.abs(got[layout][0] - got["padded"][0])) <= 1e-12 * np.max(np.abs(ref["Ei"]))
        assert np.max(np.abs(got[layout][1] - got["padded"][1])) <= 1e-12 * np.max(np.abs(ref["F"]))


@pytest.mark.parametrize("sizes", [(4, 7, 4), (5,) * 20, (4, 12)])
def test_batches_match_single_structures(sizes):
    import torch

    boxes = [synth.water_box(s, 40 + i) for i, s in enumerate(sizes)]
    pot = make_potential("fp64")
    pos = torch.tensor(np.concatenate([b.pos for b in boxes]), device="cuda")
    types = torch.tensor(np.concatenate([b.types for b in boxes]), dtype=torch.int32, device="cuda")
    offs = np.cumsum([0] + [b.n_atoms for b in boxes])
    say("neighbour split batch", sizes)
    for _ in range(2):
        _, ei, f = pot.compute_batch(pos, types, offs, np.stack([b.box for b in boxes]))
        ei, f = ei.cpu().numpy(), f.cpu().numpy()
        for k, b in enumerate(boxes):
            _, ei1, f1 = run(pot, b)
            s = slice(offs[k], offs[k + 1])
            assert np.max(np.abs(ei[s] - ei1)) <= 1e-13 * np.max(np.abs(ei1))
            assert np.max(np.abs(f[s] - f1)) <= 1e-12 * max(np.max(np.abs(f1)), 1.0)
    pot.close()

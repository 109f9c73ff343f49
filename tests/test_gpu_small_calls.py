"""The launches of small calls: the one-block sort (up to 4,096 atoms and as many
(element, cell) keys) and the grid of kernels beyond it, the one-block scan of
the keys, the batch description in kernel arguments (up to 1 KB) or uploaded,
and the energies of structures of one 4,096-atom chunk, of several and of none.
FP64 against the oracle at the FP64 bars around each limit, and batches against
the same structures computed alone (1e-13)."""
import numpy as np
import pytest

from common import oracle_water
from gpu_common import check_fp64, dev, make_potential, run, say
from paper_2002_00054_amd import synth

pytestmark = pytest.mark.gpu


def _first(n, side, seed, stretch=1.0):
    """The first n atoms of a water box (its lattice stretched: more cells per atom)."""
    b = synth.water_box(side, seed, spacing=synth.WATER_SPACING * stretch)
    assert b.n_atoms >= n
    return synth.Box(pos=b.pos[:n], types=b.types[:n], box=b.box)


@pytest.mark.parametrize("n,side,stretch", [
    (1, 4, 1.0), (63, 4, 1.0), (4095, 12, 1.0), (4096, 12, 1.0), (4097, 12, 1.0), (5184, 12, 1.0),
    (4096, 12, 2.4),   # 14 cells per axis, two elements: 5,488 keys, beyond one block
    (3000, 10, 2.4),   # 12 cells per axis: 3,456 keys
])
def test_forward_around_the_one_block_limits(n, side, stretch):
    b = _first(n, side, 50 + n % 7, stretch)
    say("small calls", n, "box", b.box[0])
    ref = oracle_water().compute(b.pos, b.types, b.box, use_cells=True)
    pot = make_potential("fp64")
    for _ in range(2):  # a second call on the same workspace
        e, ei, f = run(pot, b)
        assert e == pytest.approx(ref["E"], rel=1e-9)
        if n > 1:
            check_fp64(ei, f, ref["Ei"], ref["F"])
    pot.close()


@pytest.mark.parametrize("sizes", [
    (192,), (0,), (0, 192, 0), (81,) * 8, (81,) * 9, (81,) * 10, (81,) * 40, (4096, 3), (4097, 3), (5184, 0, 4096),
])
def test_batch_equals_single_structures(sizes):
    import torch

    boxes = [_first(n, 4 if n <= 192 else 12, 70 + i) for i, n in enumerate(sizes)]
    say("small calls batch", sizes)
    pot = make_potential("fp64")
    pos = torch.tensor(np.concatenate([b.pos for b in boxes]), device=dev())
    types = torch.tensor(np.concatenate([b.types for b in boxes]), dtype=torch.int32, device=dev())
    offs = np.cumsum([0] + list(sizes))
    eb, ei, f = pot.compute_batch(pos, types, offs, np.stack([b.box for b in boxes]))
    eb, ei, f = eb.cpu().numpy(), ei.cpu().numpy(), f.cpu().numpy()
    for k, b in enumerate(boxes):
        e1, ei1, f1 = run(pot, b)
        s = slice(offs[k], offs[k + 1])
        assert abs(eb[k] - e1) <= 1e-13 * max(1.0, np.sum(np.abs(ei1)))
        if b.n_atoms:
            assert np.max(np.abs(ei[s] - ei1)) <= 1e-13 * np.max(np.abs(ei1))
            assert np.max(np.abs(f[s] - f1)) <= 1e-12 * max(np.max(np.abs(f1)), 1.0)
    pot.close()


@pytest.mark.parametrize("n", [192, 5184])
def test_errors_are_reported_by_their_call_alone(n):
    """A bad type and a non-finite coordinate are found by the sort of either
    path; the next call on the handle is sound."""
    import torch
    from paper_2002_00054_amd.nnp import NNPError

    b = _first(n, 4 if n <= 192 else 12, 5)
    pot = make_potential("fp64")
    good = run(pot, b)
    pos = torch.tensor(b.pos, device=dev())
    types = torch.tensor(b.types, dtype=torch.int32, device=dev())
    bad_t, bad_p = types.clone(), pos.clone()
    bad_t[n // 2] = 7
    bad_p[n - 1, 2] = float("nan")
    for p, t, status in ((pos, bad_t, -3), (bad_p, types, -1)):
        with pytest.raises(NNPError) as ex:
            pot.compute(p, t, b.box)
        assert ex.value.status == status
        again = run(pot, b)
        assert np.array_equal(again[1], good[1])
    pot.close()

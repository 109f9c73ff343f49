"""The weight-gradient pass at the edges of its chunks (64 atoms of one element,
eight per round) and of its reduction (eight running sums over the chunks): from
one atom of an element to several chunks, elements without atoms, structures
without atoms among others, no dL/dE, no dL/dF. FP64 against the oracle's gradient
per tensor (1e-8), the two parts against their sum (1e-12: the sums' order is
fixed), FP32 against FP64 (2e-4)."""
import numpy as np
import pytest

import oracle
from common import water_potential
from gpu_common import dev, gpu_loss_and_grad, make_potential, per_tensor_rel, say
from paper_2002_00054_amd import synth

pytestmark = pytest.mark.gpu


def _atoms(n_h, n_o, seed):
    """n_h + n_o atoms of a water box (in a box of their own)."""
    b = synth.water_box(8, seed)
    h, o = np.nonzero(b.types == 0)[0][:n_h], np.nonzero(b.types == 1)[0][:n_o]
    k = np.sort(np.concatenate([h, o]))
    return synth.Box(pos=b.pos[k], types=b.types[k], box=b.box)


def _grad(form, boxes, gE, gF):
    import torch

    pot = make_potential(form)
    pos = torch.tensor(np.concatenate([b.pos for b in boxes]), dtype=pot.dtype, device=dev())
    types = torch.tensor(np.concatenate([b.types for b in boxes]), dtype=torch.int32, device=dev())
    offs = np.cumsum([0] + [b.n_atoms for b in boxes])
    bx = np.stack([b.box for b in boxes])
    gE = None if gE is None else torch.tensor(gE, device=dev())
    gF = None if gF is None else torch.tensor(gF, device=dev())
    g = pot.backward(pos, types, offs, bx, gE, gF).cpu().numpy()
    again = pot.backward(pos, types, offs, bx, gE, gF).cpu().numpy()  # on the kept list, launched ahead
    pot.close()
    assert np.array_equal(g, again)
    return g


@pytest.mark.parametrize("counts", [
    [(1, 0)], [(0, 1)], [(7, 1)], [(8, 9)], [(63, 64)], [(65, 128)], [(129, 0)], [(600, 300)],
    [(40, 20), (25, 44), (1, 0)],
])
def test_gradient_around_the_chunk_edges(counts):
    boxes = [_atoms(h, o, 3 + i) for i, (h, o) in enumerate(counts)]
    n = sum(b.n_atoms for b in boxes)
    say("wgrad chunks", counts)
    table, nets = water_potential()
    teacher = oracle.Potential(table, synth.xavier_nets(synth.sf_counts(table, 2), 77))
    Ehat, Fhat = oracle.batch_energy_forces(teacher, boxes)
    _, ref = oracle.loss_and_grad(oracle.Potential(table, nets), boxes, Ehat, Fhat)
    pot = make_potential("fp64")
    _, g = gpu_loss_and_grad(pot, boxes, Ehat, Fhat, synth.flat_params(nets))
    pot.close()
    assert per_tensor_rel(g, ref, nets).max() < 1e-8
    # the two parts, with an empty structure between the others
    rng = np.random.default_rng(n)
    gE, gF = rng.standard_normal(len(boxes)), rng.standard_normal((n, 3))
    both = _grad("fp64", boxes, gE, gF)
    empty = synth.Box(pos=np.zeros((0, 3)), types=np.zeros(0, dtype=np.int32), box=boxes[0].box)
    parts = _grad("fp64", [empty] + boxes + [empty], np.concatenate([[9.0], gE, [9.0]]), None) + _grad("fp64", boxes, None, gF)
    assert np.max(np.abs(parts - both)) <= 1e-12 * np.max(np.abs(both))
    assert np.linalg.norm(_grad("fp32", boxes, gE, gF) - both) <= 2e-4 * np.linalg.norm(both)

"""A gradient call takes its rows and level from its own batch, whatever the handle saw
before.  A first call on a ball of atoms, each with some 430 neighbours, leaves the
capacity that the next forward is launched with; an FP64 force-adjoint pass of that
capacity does not fit the LDS at one wave per centre, while the SF and force passes
do.  The gradient of an ordinary batch is that of a handle of its own, bit for bit (the
same kernels on the same rows; every sum has a fixed order)."""
import numpy as np
import pytest

from gpu_common import dev, make_potential, run, say
from paper_2002_00054_amd import synth

pytestmark = pytest.mark.gpu


def _ball():
    g = np.arange(-3.0, 3.0, 0.616)
    pts = np.array([(x, y, z) for x in g for y in g for z in g]) + 0.3
    pts = pts[np.einsum("ij,ij->i", pts, pts) <= 2.9 ** 2]
    pts = pts + np.random.default_rng(3).uniform(-0.04, 0.04, pts.shape)
    types = np.where(np.arange(len(pts)) % 3 == 0, synth.O, synth.H).astype(np.int32)
    return synth.Box(pos=pts + 7.0, types=types, box=np.array([14.0, 14.0, 14.0]))


@pytest.mark.parametrize("level", ["auto", "wave"])
@pytest.mark.parametrize("side", [5, 9])  # 375 and 2,187 atoms: two waves and one per centre under auto
def test_gradient_after_a_denser_call(level, side):
    import torch

    ball = _ball()
    assert 416 <= ball.n_atoms - 1 <= 456
    b = synth.water_box(side, 12)
    pos = torch.tensor(b.pos, device=dev())
    types = torch.tensor(b.types, dtype=torch.int32, device=dev())
    rng = np.random.default_rng(2)
    dE = torch.tensor(rng.standard_normal(1), device=dev())
    dF = torch.tensor(rng.standard_normal((b.n_atoms, 3)), device=dev())
    grads = []
    for first in (None, ball):
        pot = make_potential("fp64")
        pot.set_parallelism(level)
        say("row capacity", level, b.n_atoms, "after", first.n_atoms if first is not None else None)
        run(pot, first if first is not None else b)
        pot.compute_batch(pos, types, [0, b.n_atoms], [b.box])
        grads.append(pot.backward(pos, types, [0, b.n_atoms], [b.box], dE, dF).cpu().numpy())
        pot.close()
    assert np.array_equal(grads[0], grads[1])

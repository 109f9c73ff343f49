"""A handle's second and later calls launch every pass behind the neighbour
build before the host has seen its flags. Each sequence here runs on one
handle, and every result has to be that of a handle of its own: energies bitwise
(the descriptors and networks do not depend on the row capacity), forces up to
the order of the FP64 sums (1e-12 of the largest in FP64; 1e-5 eV/A in FP32,
whose forces are stored in FP32).

Row counts that outgrow the capacity of the last call by less and by more than
the list's, sizes at both numbers of waves per centre, errors between good
calls (the outputs stay untouched), batches, and gradients whose inputs differ
from the last forward's."""
import numpy as np
import pytest

from gpu_common import dev, make_potential, run, say
from paper_2002_00054_amd import synth

pytestmark = pytest.mark.gpu


def _box(side, seed, squeeze=1.0):
    """A water box, squeezed: more neighbours per atom."""
    return synth.water_box(side, seed, spacing=synth.WATER_SPACING * squeeze)


def _alone(form, b, prep=None):
    pot = make_potential(form)
    if prep:
        prep(pot)
    out = run(pot, b)
    pot.close()
    return out


def _same(form, got, ref):
    assert got[0] == ref[0] and np.array_equal(got[1], ref[1])
    tol = 1e-12 * max(np.max(np.abs(ref[2])), 1.0) if form == "fp64" else 1e-5 * max(np.max(np.abs(ref[2])), 1.0)
    assert np.max(np.abs(got[2] - ref[2])) <= tol


@pytest.mark.parametrize("layout", ["padded", "index"])
@pytest.mark.parametrize("form", ["fp64", "fp32", "bf16"])
@pytest.mark.parametrize("side", [6, 9, 12])  # 648 and 2,187 atoms around the change to one wave per centre, 5,184
def test_rows_that_grow_and_shrink(form, side, layout):
    prep = lambda p: p.set_list_layout(layout)
    boxes = [_box(side, 3 + i, q) for i, q in enumerate((1.0, 1.0, 0.97, 0.8, 1.0, 0.9, 1.3, 1.25, 0.7))]
    pot = make_potential(form)
    prep(pot)
    for i, b in enumerate(boxes):
        say("ahead", form, layout, b.n_atoms, "call", i)
        _same(form, run(pot, b), _alone(form, b, prep))
    pot.close()


@pytest.mark.parametrize("side", [4, 12])
def test_a_clustered_box_overflows_the_list(side):
    """All atoms in an eighth of the box: rows far beyond the mean density's capacity."""
    b = _box(side, 8)
    c = synth.Box(pos=b.pos * 0.5, types=b.types, box=b.box)
    pot = make_potential("fp64")
    for x in (b, b, c, b, c):
        say("ahead clustered", x.n_atoms)
        _same("fp64", run(pot, x), _alone("fp64", x))
    pot.close()


@pytest.mark.parametrize("side", [4, 12])
def test_errors_leave_the_outputs_untouched(side):
    import torch
    from paper_2002_00054_amd.nnp import NNPError

    b = _box(side, 5)
    n = b.n_atoms
    pot = make_potential("fp64")
    pos = torch.tensor(b.pos, device=dev())
    types = torch.tensor(b.types, dtype=torch.int32, device=dev())
    ei, f = torch.empty(n, dtype=torch.float64, device=dev()), torch.empty(n, 3, dtype=torch.float64, device=dev())
    good = None
    bad_t, bad_p = types.clone(), pos.clone()
    bad_t[n // 2] = 7
    bad_p[n - 1, 2] = float("nan")
    for p, t, status in ((pos, types, 0), (pos, types, 0), (pos, bad_t, -3), (bad_p, types, -1), (pos, types, 0)):
        ei.fill_(-3.0)
        f.fill_(-5.0)
        if status == 0:
            e = pot.compute_noalloc(p, t, b.box, ei, f) if n <= 1029 else None
            if e is None:
                e, ei, f = pot.compute(p, t, b.box)
            torch.cuda.synchronize()
            if good is None:
                good = (e, ei.cpu().numpy().copy(), f.cpu().numpy().copy())
            _same("fp64", (e, ei.cpu().numpy(), f.cpu().numpy()), good)
        elif n <= 1029:
            with pytest.raises(NNPError) as ex:
                pot.compute_noalloc(p, t, b.box, ei, f)
            torch.cuda.synchronize()
            assert ex.value.status == status
            assert bool((ei == -3.0).all()) and bool((f == -5.0).all())
        else:
            with pytest.raises(NNPError) as ex:
                pot.compute(p, t, b.box)
            assert ex.value.status == status
    pot.close()


@pytest.mark.parametrize("layout", ["padded", "index", "compact"])
def test_gradients_after_a_forward_of_other_inputs(layout):
    """backward on the last forward's inputs, on moved positions, on exchanged
    types, on a denser batch, and again on the first: each as a handle of its own
    gives it (FP64; the gradient's sums have a fixed order, 1e-12)."""
    import torch

    pot = make_potential("fp64")
    pot.set_list_layout(layout)
    rng = np.random.default_rng(4)

    def batch(squeeze, seed):
        bs = [_box(s, seed + s, squeeze) for s in (5, 6)]
        return (torch.tensor(np.concatenate([b.pos for b in bs]), device=dev()),
                torch.tensor(np.concatenate([b.types for b in bs]), dtype=torch.int32, device=dev()),
                np.cumsum([0] + [b.n_atoms for b in bs]), np.stack([b.box for b in bs]))

    p0, t0, offs, bx = batch(1.0, 20)
    p1, t1, offs1, bx1 = batch(0.8, 30)
    p2 = p0.clone()
    p2[7, 1] += 0.25
    t2 = t0.flip(0).contiguous()
    dE = torch.tensor(rng.standard_normal(2), device=dev())
    dF = torch.tensor(rng.standard_normal((p0.shape[0], 3)), device=dev())

    def alone(args):
        q = make_potential("fp64")
        g = q.backward(*args, dL_dE=dE, dL_dF=dF).clone()
        q.close()
        return g

    pot.compute_batch(p0, t0, offs, bx)
    for k, args in enumerate([(p0, t0, offs, bx), (p2, t0, offs, bx), (p2, t2, offs, bx), (p1, t1, offs1, bx1),
                              (p0, t0, offs, bx), (p0, t0, offs, bx)]):
        say("ahead backward", layout, k)
        g, r = pot.backward(*args, dL_dE=dE, dL_dF=dF), alone(args)
        assert torch.max(torch.abs(g - r)) <= 1e-12 * torch.max(torch.abs(r))
    pot.close()

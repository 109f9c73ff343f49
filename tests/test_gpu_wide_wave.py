"""Wide angular functions at one wave per centre against the thread-per-centre
passes (two walks of the pairs and formulas of their own): energies and forces
in FP64 (1e-12 relative) and FP32 (the oracle bars doubled: each side is within
one of them), and the weight gradient (1e-11), over tables whose classes are all
wide, mixed narrow and wide, wide in some classes only, and of four angular
eta; boxes down to two cells per axis and an empty one.  A table that gives one
wide SF twice, and an atom with more neighbours than a wave stages, keep to the
thread level and still match it."""
import numpy as np
import pytest

import oracle
from gpu_common import make_potential, oracle_input, run, say
from paper_2002_00054_amd import synth

pytestmark = pytest.mark.gpu

H, O = synth.H, synth.O


def _water(kinds, etas=(0.001, 0.03), twice=False):
    """Radial SFs and, per class, the kinds given for it."""
    t = []
    for c in (H, O):
        for nb in (H, O):
            t += [synth.SF(c, 2, (nb,), eta, shift=4.0, scale=4.0) for eta in synth.RADIAL_ETAS[:4]]
        for cls, ks in zip(synth.PAIR_CLASSES, kinds):
            for kind in ks:
                for i, eta in enumerate(etas):
                    t.append(synth.SF(c, kind, cls, eta, 0.0, (1.0, 4.0, 2.0, 16.0)[i], (-1.0, 1.0)[i % 2],
                                      shift=20.0, scale=40.0))
        if twice:
            t.append(synth.SF(c, 9, (H, H), etas[0], 0.0, 1.0, -1.0, shift=20.0, scale=40.0))
    return t, synth.xavier_nets(synth.sf_counts(t), 19)


TABLES = {
    "fcc": lambda: (synth.ni_table_scaled(wide=True), synth.ni_nets()),
    "wide": lambda: _water(((9,), (9,), (9,))),
    "mixed": lambda: _water(((3, 9), (3, 9), (3, 9))),
    "some": lambda: _water(((3,), (9,), ())),
    "four_eta": lambda: _water(((9,), (3,), (9,)), etas=(0.001, 0.01, 0.03, 0.06)),
    "twice": lambda: _water(((3, 9), (9,), (3,)), twice=True),
}


def _boxes(name):
    if name == "fcc":
        return [synth.fcc_box(3, 1), synth.fcc_box(5, 2)]
    return [synth.water_box(4, 3), synth.water_box(5, 4)]


def _both(form, table, nets, b):
    out = []
    for level in ("auto", "thread"):
        pot = make_potential(form, table, nets)
        pot.set_parallelism(level)
        out.append(run(pot, b))
        pot.close()
    return out


def _agree(form, new, old):
    (e1, ei1, f1), (e0, ei0, f0) = new, old
    if form == "fp64":
        assert np.max(np.abs(ei1 - ei0)) <= 1e-12 * np.max(np.abs(ei0))
        assert np.max(np.abs(f1 - f0)) <= 1e-12 * np.max(np.abs(f0))
    else:
        assert np.max(np.abs(ei1 - ei0)) <= 2e-5
        assert np.max(np.abs(f1 - f0)) <= 2e-4


@pytest.mark.parametrize("form", ["fp64", "fp32"])
@pytest.mark.parametrize("name", list(TABLES))
def test_forward_agrees_with_thread_level(name, form):
    table, nets = TABLES[name]()
    for b in _boxes(name):
        say("wide", name, form, b.n_atoms)
        _agree(form, *_both(form, table, nets, b))


@pytest.mark.parametrize("name", list(TABLES))
def test_weight_gradient_agrees_with_thread_level(name):
    import torch

    table, nets = TABLES[name]()
    boxes = _boxes(name)
    rng = np.random.default_rng(6)
    pos = np.concatenate([b.pos for b in boxes])
    types = np.concatenate([b.types for b in boxes]).astype(np.int32)
    offs = np.cumsum([0] + [b.n_atoms for b in boxes])
    bx = np.stack([b.box for b in boxes])
    gE, gF = rng.normal(size=len(boxes)), rng.normal(size=pos.shape)
    grads = []
    for level in ("auto", "thread"):
        pot = make_potential("fp64", table, nets)
        pot.set_parallelism(level)
        x, t = torch.tensor(pos, device="cuda"), torch.tensor(types, device="cuda")
        g = pot.backward(x, t, offs, bx, torch.tensor(gE, device="cuda"), torch.tensor(gF, device="cuda"))
        grads.append(g.cpu().numpy())
        pot.close()
    say("wide", name, "weight gradient")
    assert np.linalg.norm(grads[0] - grads[1]) <= 1e-11 * np.linalg.norm(grads[1])


@pytest.mark.parametrize("form", ["fp64", "fp32"])
def test_dense_ball_and_empty_box(form):
    """~580 atoms all within rc of each other: beyond the LDS of one wave per
    centre in FP64.  (Every force is a sum of 1.7e5 terms: FP32 to 1e-2 of the
    rms force.)"""
    g = np.arange(-2.9, 2.9001, 0.56)
    pts = np.array([(x, y, z) for x in g for y in g for z in g])
    pts = pts[np.einsum("ij,ij->i", pts, pts) <= 2.9 ** 2]
    pts = pts + np.random.default_rng(23).uniform(-0.04, 0.04, pts.shape)
    types = np.where(np.arange(len(pts)) % 3 == 0, O, H).astype(np.int32)
    b = synth.Box(pos=pts + 7.0, types=types, box=np.array([14.0, 14.0, 14.0]))
    table, nets = TABLES["mixed"]()
    say("wide dense ball", form, b.n_atoms)
    (e1, ei1, f1), (e0, ei0, f0) = _both(form, table, nets, b)
    if form == "fp32":
        # the thread level adds an SF's 1.7e5 terms one after the other in FP32,
        # which alone moves E_i by 1e-3 of their rms: the oracle is the measure
        ref = oracle.Potential(table, nets).compute(oracle_input(b, form), b.types, b.box)
        say("thread level max dE_i/rms", np.max(np.abs(ei0 - ref["Ei"])) / np.sqrt(np.mean(ref["Ei"] ** 2)),
            "wave", np.max(np.abs(ei1 - ref["Ei"])) / np.sqrt(np.mean(ref["Ei"] ** 2)))
        ei0, f0 = ref["Ei"], ref["F"]
    rms_e, rms_f = np.sqrt(np.mean(ei0 ** 2)), np.sqrt(np.mean(f0 ** 2))
    tol_e, tol_f = (1e-11, 1e-10) if form == "fp64" else (1e-4, 1e-2)
    assert np.max(np.abs(ei1 - ei0)) <= tol_e * rms_e
    assert np.max(np.abs(f1 - f0)) <= tol_f * max(rms_f, 1e-3)
    empty = synth.Box(pos=np.zeros((0, 3)), types=np.zeros(0, dtype=np.int32), box=b.box)
    pot = make_potential(form, table, nets)
    e, ei, f = run(pot, empty)
    pot.close()
    assert e == 0.0 and ei.shape == (0,) and f.shape == (0, 3)

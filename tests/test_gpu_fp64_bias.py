"""FP64 symmetry functions summed over a box carry no common error.

Energies are differences of large sums of symmetry-function terms, so an error that
every term shares (a rounded constant in the cutoff's argument, say) reaches the
energy of a box multiplied by that cancellation, however small it is in one term.
A network whose every weight is a power of two, 2^-50 before the two tanh and 2^50
after, hands out one symmetry function as the atomic energy (tanh x = x at this
size).  Its sum over the box against numpy's extended precision: the roundings of
single terms average out over 10^4 to 10^6 different terms, and what is left is to be
within one unit roundoff (2^-53), the rounding of a single product.  Radial functions,
narrow angular ones on either side of the rules for the polynomials of the exponents
(by density: below it at 3.9 A; by exponent: 0.1), wide ones, at three cutoff radii."""
import numpy as np
import pytest

from gpu_common import make_potential, run, say
from paper_2002_00054_amd import synth

pytestmark = pytest.mark.gpu
L = np.longdouble
PI = L("3.14159265358979323846264338327950288")


def _fc(s, rc):
    return (1 + np.cos(PI * np.sqrt(s) / L(rc))) / 2


def _reference(b, rc, kind, eta, lam):
    """Sum over all centres in extended precision, terms in extended precision."""
    pos, box = b.pos.astype(L), b.box.astype(L)
    total = L(0)
    for i in range(b.n_atoms):
        d = pos - pos[i]
        d -= box * np.round(d / box)
        s = (d * d).sum(1)
        near = (s < L(rc) * L(rc)) & (np.arange(b.n_atoms) != i)
        d, s = d[near], s[near]
        g = np.exp(-L(eta) * s) * _fc(s, rc)
        if kind == 2:
            total += g.sum()
            continue
        j, k = np.triu_indices(len(s), 1)
        r = np.sqrt(s)
        cos = (d[j] * d[k]).sum(1) / (r[j] * r[k])
        t = g[j] * g[k] * (1 + L(lam) * cos)
        if kind == 3:
            sjk = ((d[j] - d[k]) ** 2).sum(1)
            t = np.where(sjk < L(rc) * L(rc), t * np.exp(-L(eta) * sjk) * _fc(sjk, rc), L(0))
        total += t.sum()
    return total


def _gas():
    """512 atoms of one element on a jittered lattice: no two distances alike."""
    rng = np.random.default_rng(17)
    a = 2.153  # water's density of atoms; the edge exceeds 12 A
    i = np.stack(np.meshgrid(*3 * [np.arange(8.0)], indexing="ij"), -1).reshape(-1, 3)
    pos = (a * (i + 0.5) + rng.uniform(-0.6, 0.6, (512, 3))) % (8 * a)
    return synth.Box(pos=pos, types=np.zeros(512, dtype=np.int32), box=np.full(3, 8 * a))


def _common_error(rc, kind, eta, lam, form):
    from paper_2002_00054_amd.nnp import Potential

    b = _gas()
    if kind == 2:
        table = [synth.SF(0, 2, (0,), eta, rc=rc)]
    else:
        table = [synth.SF(0, kind, (0, 0), eta, 0.0, 1.0, float(lam), rc=rc)]
    one, zero = np.ones((1, 1)), np.zeros(1)
    net = synth.Net(W=[one * 2.0 ** -50, one, one * 2.0 ** 50], b=[zero, zero, zero])
    pot = Potential(table, [net], precision="fp64", elements=("A",))
    if form == "stored":
        pot.set_derivative_mode("stored")
    else:
        pot.set_parallelism(form)
    _, ei, _ = run(pot, b)
    pot.close()
    ref = _reference(b, rc, kind, eta, lam)
    off = float((ei.astype(L).sum() - ref) / ref)
    say("common error", rc, kind, eta, form, "%.2e" % off)
    return off


@pytest.mark.parametrize("rc", [6.0, 5.0, 3.9])
@pytest.mark.parametrize("kind,eta,lam", [(2, 0.0, 0), (2, 0.02, 0), (3, 0.001, 1), (3, 0.03, -1), (3, 0.1, 1), (9, 0.01, -1)])
def test_sums_carry_no_common_error(rc, kind, eta, lam):
    assert abs(_common_error(rc, kind, eta, lam, "wave")) <= 2.0 ** -53


@pytest.mark.parametrize("form", ["wave2", "thread", "stored"])
@pytest.mark.parametrize("kind,eta,lam", [(2, 0.02, 0), (3, 0.03, -1)])
def test_every_form(kind, eta, lam, form):
    assert abs(_common_error(6.0, kind, eta, lam, form)) <= 2.0 ** -53


def _water_energy(b, real):
    """Total energy of a water box with the formulas evaluated in the given type."""
    table, nets = synth.water_table_scaled(), synth.water_nets()
    pos, box, rc, pi = b.pos.astype(real), b.box.astype(real), real(synth.RCUT), real(PI)
    total = real(0)
    for i in range(b.n_atoms):
        d = pos - pos[i]
        d -= box * np.round(d / box)
        s = (d * d).sum(1)
        near = (s < rc * rc) & (np.arange(b.n_atoms) != i)
        d, s, t = d[near], s[near], b.types[near]
        r = np.sqrt(s)
        fc = (1 + np.cos(pi * r / rc)) / 2
        j, k = np.triu_indices(len(s), 1)
        sjk = ((d[j] - d[k]) ** 2).sum(1)
        on = sjk < rc * rc
        j, k, sjk = j[on], k[on], sjk[on]
        cos = (d[j] * d[k]).sum(1) / (r[j] * r[k])
        f3 = fc[j] * fc[k] * (1 + np.cos(pi * np.sqrt(sjk) / rc)) / 2
        radial = {e: f3 * np.exp(-real(e) * (s[j] + s[k] + sjk)) for e in {x.eta for x in table if x.kind == 3}}
        g = []
        for x in (x for x in table if x.centre == b.types[i]):
            if x.kind == 2:
                v = (np.exp(-real(x.eta) * (r - real(x.rs)) ** 2) * fc)[t == x.nbr[0]].sum()
            else:
                e1, e2 = x.nbr
                of = ((t[j] == e1) & (t[k] == e2)) | ((t[j] == e2) & (t[k] == e1))
                v = (radial[x.eta] * (1 + real(x.lam) * cos) ** int(x.zeta))[of].sum() * real(2) ** (1 - real(x.zeta))
            g.append((v - real(x.shift)) / real(x.scale))
        a, net = np.array(g), nets[b.types[i]]
        for layer, (W, bias) in enumerate(zip(net.W, net.b)):
            a = (W.astype(real) * a).sum(1) + bias.astype(real)
            a = np.tanh(a) if layer < 2 else a
        total += a[0]
    return total


@pytest.mark.parametrize("side,seed", [(4, 35), (5, 32)])
def test_energy_is_nearer_than_plain_float64(side, seed):
    """The float64 formulas round pi and r / rc, which moves every fc the same way: their
    energy is no measure of an error of 1e-14.  Extended precision is, and the library
    is to be nearer to it than they are."""
    b = synth.water_box(side, seed)
    ref, plain = _water_energy(b, L), _water_energy(b, np.float64)
    pot = make_potential("fp64")
    _, ei, _ = run(pot, b)
    pot.close()
    off = float((ei.astype(L).sum() - ref) / ref)
    off_plain = float((L(plain) - ref) / ref)
    say("energy", b.n_atoms, "off by %.1e, plain float64 by %.1e" % (off, off_plain))
    assert abs(off) < abs(off_plain)

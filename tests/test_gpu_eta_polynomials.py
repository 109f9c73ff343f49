"""The FP64 passes on either side of the rule that chooses how they evaluate
fc(r_jk) e^{-eta r_jk^2}: as one polynomial per angular eta while eta rc^2 is
small enough for its degree (two degrees), as a cutoff polynomial times an
exponential otherwise.  The water model with its second angular eta replaced,
from far below the low degree's range to far above the high one's (eta = 0
included), against the FP64 oracle at the FP64 bars (1e-9 relative), energies
and forces at one and two waves per centre, and the weight gradient (1e-8 per
tensor) for a table on each path."""
import numpy as np
import pytest

import oracle
from gpu_common import check_fp64, gpu_loss_and_grad, make_potential, per_tensor_rel, run, say
from paper_2002_00054_amd import synth

pytestmark = pytest.mark.gpu


def _potential(eta):
    t = synth.water_table_scaled()
    for s in t:
        if s.kind == 3 and s.eta == 0.03:
            s.eta = eta
    return t, synth.water_nets()


@pytest.mark.parametrize("eta", [0.0, 0.0011, 0.0016, 0.02, 0.036, 0.039, 0.06, 0.5])
@pytest.mark.parametrize("level", ["wave", "wave2"])
def test_forward_matches_oracle(eta, level):
    table, nets = _potential(eta)
    b = synth.water_box(5, 31)
    ref = oracle.Potential(table, nets).compute(b.pos, b.types, b.box)
    say("eta", eta, level)
    pot = make_potential("fp64", table, nets)
    pot.set_parallelism(level)
    e, ei, f = run(pot, b)
    pot.close()
    check_fp64(ei, f, ref["Ei"], ref["F"])


@pytest.mark.parametrize("eta", [0.036, 0.06])
def test_weight_gradient_matches_oracle(eta):
    table, nets = _potential(eta)
    boxes = [synth.water_box(4, 33), synth.water_box(5, 34)]
    rng = np.random.default_rng(8)
    Ehat = rng.normal(size=2)
    Fhat = rng.normal(size=(sum(b.n_atoms for b in boxes), 3))
    _, ref = oracle.loss_and_grad(oracle.Potential(table, nets), boxes, Ehat, Fhat)
    say("eta", eta, "weight gradient")
    pot = make_potential("fp64", table, nets)
    L, g = gpu_loss_and_grad(pot, boxes, Ehat, Fhat, synth.flat_params(nets))
    pot.close()
    assert np.all(per_tensor_rel(g, ref, nets) <= 1e-8)

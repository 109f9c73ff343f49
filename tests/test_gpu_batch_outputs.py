"""What calls write into the caller's buffers, through the C entry points.

Energies of batches whose structures take several 16,384-atom chunks next to others
and to empty ones: each is the sum of its own atomic energies (1e-14 of the sum of
their magnitudes: FP64 tree sums of some 2^15 terms).  And calls that are refused only
after their passes have been launched (second calls on a handle, 5,184 atoms): device
energies, atomic energies, forces and gradient stay as the caller left them."""
import ctypes as C

import numpy as np
import pytest

from gpu_common import dev, make_potential, say
from paper_2002_00054_amd import synth

pytestmark = pytest.mark.gpu


class Call:
    """A batch and buffers of the caller's for its outputs."""

    def __init__(self, pot, boxes, sizes):
        import torch

        self.pot, self.torch = pot, torch
        self.pos = torch.tensor(np.concatenate([b.pos[:n] for b, n in zip(boxes, sizes)]), device=dev())
        self.types = torch.tensor(np.concatenate([b.types[:n] for b, n in zip(boxes, sizes)]), dtype=torch.int32, device=dev())
        self.offs = np.cumsum([0] + list(sizes)).astype(np.int64)
        self.box = np.ascontiguousarray(np.stack([b.box for b in boxes]))
        n, k = len(self.types), len(sizes)
        new = lambda *s: torch.full(s, -7.5, dtype=torch.float64, device=dev())
        self.e, self.ei, self.f, self.grad = new(k), new(n), new(n, 3), new(pot.n_params)
        self.gE, self.gF = torch.ones(k, dtype=torch.float64, device=dev()), torch.ones(n, 3, dtype=torch.float64, device=dev())

    def _args(self, pos, types):
        return (self.pot._h, len(self.box), self.offs.ctypes.data_as(C.POINTER(C.c_int64)), pos.data_ptr(),
                types.data_ptr(), self.box.ctypes.data_as(C.POINTER(C.c_double)))

    def forward(self, pos=None, types=None):
        st = self.pot._L.nnp_compute_batch(*self._args(self.pos if pos is None else pos, self.types if types is None else types),
                                           self.e.data_ptr(), self.ei.data_ptr(), self.f.data_ptr(),
                                           self.torch.cuda.current_stream().cuda_stream)
        self.torch.cuda.synchronize()
        return st

    def backward(self, pos=None, types=None):
        st = self.pot._L.nnp_backward(*self._args(self.pos if pos is None else pos, self.types if types is None else types),
                                      self.gE.data_ptr(), self.gF.data_ptr(), self.grad.data_ptr(),
                                      self.torch.cuda.current_stream().cuda_stream)
        self.torch.cuda.synchronize()
        return st

    def fill(self):
        for x in (self.e, self.ei, self.f, self.grad):
            x.fill_(-7.5)
        self.torch.cuda.synchronize()

    def untouched(self):
        return all(bool((x == -7.5).all()) for x in (self.e, self.ei, self.f, self.grad))


@pytest.mark.parametrize("sizes", [(16385, 0, 192), (192, 32769, 3), (0, 16384, 16385, 81)])
def test_energies_of_several_chunks_in_a_batch(sizes):
    pot = make_potential("fp64")
    c = Call(pot, [synth.water_box(23 if n > 192 else 4, 40 + i) for i, n in enumerate(sizes)], sizes)
    for call in range(2):
        say("chunks", sizes, "call", call)
        c.fill()
        assert c.forward() == 0
        e, ei = c.e.cpu().numpy(), c.ei.cpu().numpy()
        for k in range(len(sizes)):
            own = ei[c.offs[k]:c.offs[k + 1]]
            assert abs(e[k] - np.sum(own.astype(np.longdouble))) <= 1e-14 * np.sum(np.abs(own))
    pot.close()


@pytest.mark.parametrize("bad", ["type", "nan"])
def test_refused_calls_leave_the_buffers(bad):
    pot = make_potential("fp64")
    c = Call(pot, [synth.water_box(12, 9)], (5184,))
    pos, types = c.pos.clone(), c.types.clone()
    if bad == "type":
        types[2000] = 7
    else:
        pos[5183, 1] = float("nan")
    status = -3 if bad == "type" else -1
    assert c.forward() == 0 and c.backward() == 0
    for call in range(2):  # with a forward to reuse, and with none
        say("refused", bad, "call", call)
        c.fill()
        assert c.backward(pos, types) == status and c.untouched()
        assert c.forward(pos, types) == status and c.untouched()
    assert c.forward() == 0 and c.backward() == 0 and not bool((c.grad == -7.5).any())
    pot.close()

"""What a handle keeps between calls, on the CPU: the built library over a stand-in for
the HIP runtime (fake_hip.cpp), in a process of its own.

nnp_backward reuses the last batch forward if its inputs are the same, which a kernel
compares while the gradient's kernels are already launched behind a gate.  After a call
that failed between the two, a gradient on the first inputs is written, whether it
reuses the forward or repeats it."""
import os
import subprocess
import sys

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))

PROGRAM = r"""
import ctypes as C, sys, types
sys.path[:0] = [sys.argv[2], sys.argv[3]]
sys.modules["torch"] = types.ModuleType("torch")  # would load the real runtime
fake = C.CDLL(sys.argv[1], mode=C.RTLD_GLOBAL)
fake.fake_fail_launch.argtypes = fake.fake_launches.argtypes = [C.c_char_p]
fake.fake_launches.restype = C.c_long
import numpy as np
from paper_2002_00054_amd import nnp, synth
from common import water_potential
L = nnp.load_library()
pot = nnp.Potential(*water_potential(), precision="fp64")

class Batch:
    def __init__(self, side, seed, stretch=1.0):
        b = synth.water_box(side, seed, spacing=synth.WATER_SPACING * stretch)
        self.n, self.pos, self.types = b.n_atoms, b.pos.copy(), b.types.astype(np.int32)
        self.offs, self.box = (C.c_int64 * 2)(0, b.n_atoms), (C.c_double * 3)(*b.box)
    def args(self):
        return (pot._h, 1, self.offs, self.pos.ctypes.data, self.types.ctypes.data, self.box)
    def forward(self):
        e, ei, f = np.zeros(1), np.zeros(self.n), np.zeros((self.n, 3))
        return L.nnp_compute_batch(*self.args(), e.ctypes.data, ei.ctypes.data, f.ctypes.data, None)
    def backward(self):
        g, dE, dF = np.zeros(pot.n_params), np.ones(1), np.ones((self.n, 3))
        st = L.nnp_backward(*self.args(), dE.ctypes.data, dF.ctypes.data, g.ctypes.data, None)
        return st, bool((g == 1.0).all())

a, other, larger = Batch(5, 1), Batch(5, 2), Batch(6, 3)
sorts = lambda: fake.fake_launches(b"k_sort_small")
assert a.forward() == 0 and a.forward() == 0
n = sorts()
assert a.backward() == (0, True) and sorts() == n  # the forward is reused
"""


@pytest.fixture(scope="module")
def fake(tmp_path_factory):
    from paper_2002_00054_amd import build, nnp

    if not os.path.exists(nnp.LIB_PATH):
        build.build(verbose=False)
    so = str(tmp_path_factory.mktemp("fake") / "libamdhip64.so.7")
    subprocess.run(["g++", "-O1", "-std=c++17", "-shared", "-fPIC", "-Wl,-soname,libamdhip64.so.7", "-o", so,
                    os.path.join(HERE, "fake_hip.cpp")], check=True)
    return so


def _run(fake, more):
    r = subprocess.run([sys.executable, "-c", PROGRAM + more, fake, os.path.dirname(HERE), HERE], capture_output=True,
                       text=True, timeout=120)
    assert r.returncode == 0, r.stderr[-3000:]


FAILED = """
assert other.backward()[0] == nnp_error
n = sorts()
st, written = a.backward()
assert st == 0 and written, (st, written)
assert a.backward() == (0, True)
"""


@pytest.mark.parametrize("kernel", ["k_triplet", "k_wgrad_final"])
def test_a_launch_fails_behind_the_comparison(fake, kernel):
    _run(fake, "nnp_error = -4\nfake.fake_fail_launch(b'%s')" % kernel + FAILED)


def test_the_wait_for_the_comparison_fails(fake):
    _run(fake, "nnp_error = -4\nfake.fake_fail_event(0)" + FAILED)


@pytest.mark.parametrize("call", ["forward", "backward"])
def test_memory_runs_out_for_a_larger_batch(fake, call):
    """Whichever of its allocations fails: buffers before it have replaced the kept ones."""
    _run(fake, """
for k in range(40):
    assert a.forward() == 0
    n = sorts()
    assert a.backward() == (0, True) and sorts() == n
    fake.fake_fail_malloc(k)
    larger = Batch(6 + k % 3, 3)  # sizes in turn, so that one always needs more
    st = larger.CALL()
    st = st[0] if isinstance(st, tuple) else st
    assert st in (0, -5), st
    fake.fake_fail_malloc(-1)
    n = sorts()
    assert a.backward() == (0, True) and sorts() > n, (k, st)
""".replace("CALL", call))


def test_stages_of_a_call_whose_rows_outgrew_the_capacity(fake):
    """Its passes are run again; every stage of the call is still reported, the sort too."""
    _run(fake, """
stages = ["bin_sort", "neighbors", "sf", "mlp", "force", "finish"]
pot.set_profiling(True)
for rows in (90, 90, 110):
    fake.fake_rows(rows)
    n = fake.fake_launches(b"k_mlp")
    assert a.forward() == 0
    assert list(pot.timings()) == stages, (rows, pot.timings())
assert fake.fake_launches(b"k_mlp") == n + 2
""")


AHEAD = """
pot = nnp.Potential(*water_potential(), precision="fp64")
def forward(batch):  # whether the call launched its passes before it saw the flags
    n, m = fake.fake_launches(b"k_max_count"), fake.fake_launches(b"k_mlp")
    assert batch.forward() == 0
    return fake.fake_launches(b"k_max_count") == n, fake.fake_launches(b"k_mlp") - m
ONCE, WAITED, TWICE = (True, 1), (False, 1), (False, 2)
fake.fake_lds.restype, fake.fake_lds.argtypes = C.c_size_t, [C.c_char_p]
fake.fake_rows(100)
"""


def test_a_denser_batch_waits_for_its_rows(fake):
    _run(fake, AHEAD + """
dense = Batch(6, 4, 0.95)
assert forward(a) == WAITED and forward(a) == ONCE  # 100 rows for the first time, then known
fake.fake_rows(115)
assert forward(dense) == WAITED and forward(dense) == ONCE
fake.fake_rows(100)
assert forward(a) == ONCE and forward(dense) == ONCE  # small batches: the longer rows cost nothing
""")


def test_a_sparser_large_batch_waits_for_its_rows(fake):
    _run(fake, AHEAD + """
large, sparse = Batch(18, 5), Batch(18, 6, 1.1)
assert forward(large) == WAITED and forward(large) == ONCE
fake.fake_rows(80)
assert forward(sparse) == WAITED and forward(sparse) == ONCE
""")


def test_a_large_batch_gives_up_longer_rows_at_once(fake):
    """Rows of a clustered box (the same mean density) are kept for one call."""
    _run(fake, AHEAD + """
large = Batch(18, 5)
assert forward(large) == WAITED and forward(large) == ONCE
own = fake.fake_lds(b"k_triplet")
pot.set_list_layout("compact")  # (waits: no run ahead)
fake.fake_rows(190)
forward(large)
pot.set_list_layout("padded")
fake.fake_rows(100)
assert forward(large) == ONCE and fake.fake_lds(b"k_triplet") > own
assert forward(large) == ONCE and fake.fake_lds(b"k_triplet") == own
""")


def test_large_batches_wait_after_a_miss(fake):
    """A call whose rows outgrew the capacity pays for its passes twice: the next 16
    wait, twice as many after the next such call.  A small batch gains more by running
    ahead than a miss in 16 calls costs it."""
    _run(fake, AHEAD + """
large = Batch(18, 5)
assert forward(large) == WAITED and forward(large) == ONCE
for waits in (16, 32):
    fake.fake_rows(100 + waits // 2)
    assert forward(large) == TWICE
    for k in range(waits):
        assert forward(large) == WAITED, k
    assert forward(large) == ONCE
fake.fake_rows(100)
pot = nnp.Potential(*water_potential(), precision="fp64")
assert forward(a) == WAITED and forward(a) == ONCE
fake.fake_rows(110)
assert forward(a) == TWICE and forward(a) == ONCE
""")


def test_four_eta_tables_keep_the_exponentials(fake):
    """FP64 passes of tables with more than two angular etas: the polynomials' 60
    coefficients cost more than the exponentials they replace, at every density."""
    _run(fake, AHEAD + """
def table(etas):
    t = []
    for c in (0, 1):
        t += [synth.SF(c, 2, (nb,), 0.01) for nb in (0, 1)]
        for cls in synth.PAIR_CLASSES:
            t += [synth.SF(c, 3, cls, eta, 0.0, 2.0, 1.0) for eta in etas]
    return t, synth.xavier_nets(synth.sf_counts(t), 5)
poly = lambda: fake.fake_launches(b"Lb1ELb0EEEv")  # k_triplet<..., POLY, not WIDE>
for etas, used in (((0.001, 0.03), True), ((0.001, 0.01, 0.03), False), ((0.001, 0.01, 0.02, 0.03), False)):
    pot = nnp.Potential(*table(etas), precision="fp64")
    n, m = poly(), fake.fake_launches(b"k_triplet")
    forward(a)
    a.backward()
    assert fake.fake_launches(b"k_triplet") > m
    assert (poly() > n) == used, etas
""")

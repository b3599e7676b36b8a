"""Which calls launch passes while later ones are being planned, and what a
call that must not does with the state.  The passes are counted, so that a call
that was launched whole does not pass for one that was not."""
import numpy as np
import pytest

import oracle
from circuits import layered_circuit

torch = pytest.importorskip("torch")
from paper_2502_11385_amd import qsv  # noqa: E402

pytestmark = pytest.mark.gpu
C64, C128 = qsv.QSV_C64, qsv.QSV_C128
N = 16
MANY = layered_circuit(N, 60, 7)     # about 1400 gates, over 64 KiB of program


@pytest.fixture(autouse=True)
def _need_gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    yield
    qsv.debug_inject(1, 0)


def _warm(prec, gates=MANY, stream=None):
    """A state whose program buffer and both large staging buffers are there."""
    s = qsv.State(N, prec, stream=stream)
    circ = qsv.Circuit.from_gates(gates)
    for _ in range(2):
        s.init_basis(0)
        s.sync()
        s.apply_fused(circ)
        assert s.early_passes() == 0
    s.sync()
    return s, circ


@pytest.mark.parametrize("prec", [C64, C128])
def test_parts_give_the_oracles_state(prec):
    s, circ = _warm(prec)
    s.init_basis(0)
    s.sync()
    whole = qsv.State(N, prec)
    whole.init_basis(0)
    whole.apply_fused(circ)
    for outputs in (False, True, True):
        s.init_basis(0)
        s.sync()                     # idle: the first chance is taken
        if outputs:                  # the first such call sizes the scratch
            marg, _ = s.apply_fused_outputs(circ, marg_qubits=[0, 7, 15])
        else:
            s.apply_fused(circ)
        early, stats = s.early_passes(), s.plan_stats()
        assert stats["gates"] == len(MANY)
        assert early < stats["passes"]
        got = s.get()
        assert np.array_equal(got, whole.get())
    assert early > 0
    p = np.abs(got.astype(complex)) ** 2
    assert np.max(np.abs(marg - oracle.marginal(p, N, [0, 7, 15]))) <= (
        2e-6 if prec == C64 else 1e-12)
    want = oracle.simulate(N, MANY)
    eps = 2.0 ** -24 if prec == C64 else 2.0 ** -53
    assert np.max(np.abs(got - want)) <= 4 * eps * np.sqrt(len(MANY)) + 1e-14
    whole.free()
    s.free()


def test_parts_are_launched_without_outputs():
    s, circ = _warm(C64)
    s.init_basis(0)
    s.sync()
    s.apply_fused(circ)
    assert s.early_passes() > 0
    s.free()


# too few gates after the first passes; a program beyond the bound; below the
# width where planning takes long; a plan that is not tiled
@pytest.mark.parametrize("n,depth,opts", [
    (16, 2, None), (16, 130, None), (15, 60, None),
    (16, 60, qsv.fuse_opts(strategy=qsv.PLAN_FUSED))])
def test_other_circuits_are_launched_whole(n, depth, opts):
    s = qsv.State(n, C64)
    circ = qsv.Circuit.from_gates(layered_circuit(n, depth, 7))
    for _ in range(4):
        s.init_basis(0)
        s.sync()
        s.apply_fused(circ, opts)
        assert s.early_passes() == 0
    s.free()


def test_a_busy_stream_gets_the_circuit_whole():
    st = torch.cuda.Stream()
    s, circ = _warm(C64, stream=st)
    big = qsv.State(29, C64, stream=st)
    long = qsv.Circuit.from_gates(layered_circuit(29, 8, 1))
    big.init_basis(0)
    big.apply_fused(long)
    big.sync()
    big.apply_fused(long)            # some 10 ms; planning takes about one
    s.apply_fused(circ)
    assert s.early_passes() == 0
    big.free()
    s.free()


@pytest.mark.parametrize("prec", [C64, C128])
def test_a_failed_allocation_keeps_the_state(prec):
    """Everything for launching in parts is there but the scratch, which the
    shots need: no pass may run before its allocation is known to succeed."""
    s, circ = _warm(prec)
    s.init_basis(5)
    s.sync()
    qsv.debug_inject(1, 1)
    with pytest.raises(qsv.QsvError) as e:
        s.apply_fused_outputs(circ, shots=64)
    assert e.value.status == qsv.QSV_ERR_OUT_OF_MEMORY
    got = s.get()
    assert got[5] == 1 and np.count_nonzero(got) == 1
    s.apply_fused(circ)              # and the state still works
    assert s.early_passes() > 0
    assert abs(s.norm() - 1) < 1e-4
    s.free()

"""Single gates: states beyond 256 MiB, which are streamed past the cache, and
diagonal gates around the size where a thread takes four amplitudes
(2^18 of them under the controls): one phase and tables of one, two and five
targets, with controls on low, on high and on both kinds of qubits.

A gate multiplies each amplitude once: a few roundings of an amplitude of
modulus at most 1, 4 eps absolute."""
import numpy as np
import pytest

import oracle
from circuits import random_state

torch = pytest.importorskip("torch")
from paper_2502_11385_amd import qsv  # noqa: E402

pytestmark = pytest.mark.gpu
EPS = {qsv.QSV_C64: 2.0 ** -23, qsv.QSV_C128: 2.0 ** -52}


@pytest.fixture(scope="module", autouse=True)
def _need_gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


@pytest.mark.parametrize("prec", [qsv.QSV_C64, qsv.QSV_C128])
@pytest.mark.parametrize("n", [6, 17, 18, 19, 20])
def test_diagonal_gates(n, prec):
    rng = np.random.default_rng(n)
    s = qsv.State(n, prec)
    psi = random_state(n, n)
    if prec == qsv.QSV_C64:
        psi = psi.astype(np.complex64).astype(np.complex128)
    for k in (1, 2, 5):
        for controls in ([], [0], [n - 1], [1, n - 2]):
            free = [q for q in range(n) if q not in controls]
            if len(free) < k:
                continue
            t = [int(q) for q in rng.permutation(free)[:k]]
            for masked in (False, True):
                d = np.exp(1j * rng.uniform(0, 6.28, 1 << k))
                if masked:
                    d[:-1] = 1
                s.set(psi)
                s.apply_gate(t, np.diag(d), controls)
                want = oracle.apply_gate(psi, n, np.diag(d), t, controls)
                err = np.max(np.abs(s.get() - want))
                assert err <= 4 * EPS[prec], (k, controls, masked, err)
    s.free()


@pytest.mark.parametrize("prec,n", [(qsv.QSV_C64, 25), (qsv.QSV_C64, 26),
                                    (qsv.QSV_C128, 24), (qsv.QSV_C128, 25)])
def test_gates_around_the_streaming_size(n, prec):
    """A few gates on a basis state: the amplitudes of the qubits that took
    part, against the oracle on those qubits alone; zero elsewhere."""
    qs = [0, 3, 9, n - 1]
    rng = np.random.default_rng(n)

    def unitary(k):
        z = rng.standard_normal((2, 1 << k, 1 << k))
        return np.linalg.qr(z[0] + 1j * z[1])[0]

    gates = [([0], unitary(1), []), ([3], unitary(1), [2]),
             ([1, 3], unitary(2), []), ([2], unitary(1), []),
             ([0, 1, 2], unitary(3), []), ([3], unitary(1), [0]),
             ([3], np.diag([1, 1j]), [0]), ([1], np.diag([-1j, 1j]), []),
             ([0, 2], np.diag(np.exp(1j * rng.uniform(0, 6, 4))), [3])]
    s = qsv.State(n, prec)
    s.init_basis(0)
    want = np.zeros(16, complex)
    want[0] = 1
    for t, u, c in gates:
        s.apply_gate([qs[i] for i in t], u, [qs[i] for i in c])
        want = oracle.apply_gate(want, 4, u, t, c)
    idx = np.array([sum(1 << qs[b] for b in range(4) if x >> b & 1)
                    for x in range(16)])
    got = s.get()
    s.free()
    assert np.max(np.abs(got[idx] - want)) <= 64 * EPS[prec]
    got[idx] = 0
    assert not got.any()

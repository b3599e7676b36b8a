"""Single gates on states beyond the cache whose fixed bits leave as much as it
holds, more, or less: with and without streaming, the same gates."""
import numpy as np
import pytest

import oracle

torch = pytest.importorskip("torch")
from paper_2502_11385_amd import qsv  # noqa: E402

pytestmark = pytest.mark.gpu
EPS = {qsv.QSV_C64: 2.0 ** -23, qsv.QSV_C128: 2.0 ** -52}


@pytest.fixture(scope="module", autouse=True)
def _need_gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


@pytest.mark.parametrize("prec,n", [(qsv.QSV_C64, 26), (qsv.QSV_C64, 27),
                                    (qsv.QSV_C128, 25), (qsv.QSV_C128, 26)])
def test_controlled_gates_beyond_the_cache(n, prec):
    """A few gates on a basis state: the amplitudes of the qubits that took
    part, against the oracle on those qubits alone; zero elsewhere.  A gate
    adds a few roundings to amplitudes of modulus at most 1: 4 eps a gate."""
    qs = [1, 4, 7, 8, n - 2, n - 1]
    w = len(qs)
    rng = np.random.default_rng(n)

    def unitary(k):
        z = rng.standard_normal((2, 1 << k, 1 << k))
        return np.linalg.qr(z[0] + 1j * z[1])[0]

    def phases(k):
        return np.diag(np.exp(1j * rng.uniform(0, 6, 1 << k)))

    gates = [([q], unitary(1), []) for q in range(w)]
    for c in ([1], [2], [3], [4], [3, 5], [1, 4], [0, 3, 4]):
        free = [q for q in range(w) if q not in c]
        gates += [([free[0]], unitary(1), c), ([free[-1]], unitary(1), c),
                  (free[:2], unitary(2), c), (free[1:3], phases(2), c),
                  ([free[-1]], phases(1), c),
                  ([free[1]], np.diag([1, 1j]), c)]
    gates += [([1, 3, 5], unitary(3), []), ([0, 4, 5], unitary(3), [3])]
    s = qsv.State(n, prec)
    s.init_basis(0)
    want = np.zeros(1 << w, complex)
    want[0] = 1
    for t, u, c in gates:
        s.apply_gate([qs[i] for i in t], u, [qs[i] for i in c])
        want = oracle.apply_gate(want, w, u, t, c)
    idx = np.array([sum(1 << qs[b] for b in range(w) if x >> b & 1)
                    for x in range(1 << w)])
    got = s.get()
    s.free()
    assert np.max(np.abs(got[idx] - want)) <= 4 * len(gates) * EPS[prec]
    got[idx] = 0
    assert not got.any()

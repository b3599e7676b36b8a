"""A queue of calls that each upload something: gate matrices of 1 to 16 KiB and
programs below and above a staging buffer, in every order, so that they share
buffers, fill them and come round again while earlier ones are still read."""
import numpy as np
import pytest

import oracle
from circuits import layered_circuit, random_state

torch = pytest.importorskip("torch")
from paper_2502_11385_amd import qsv  # noqa: E402

pytestmark = pytest.mark.gpu
C64, C128 = qsv.QSV_C64, qsv.QSV_C128


@pytest.fixture(scope="module", autouse=True)
def _need_gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


@pytest.mark.parametrize("prec", [C64, C128])
@pytest.mark.parametrize("seed", [1, 2, 3])
def test_queued_uploads(seed, prec):
    n = 9
    rng = np.random.default_rng(seed)
    s = qsv.State(n, prec)
    psi = random_state(n, seed)
    s.set(psi)
    want = psi.astype(np.complex64 if prec == C64 else np.complex128)
    want = want.astype(np.complex128)
    count = 0
    for _ in range(150):
        k = int(rng.integers(0, 6))
        if k >= 3:               # a matrix of its own
            z = rng.standard_normal((2, 1 << k, 1 << k))
            u = np.linalg.qr(z[0] + 1j * z[1])[0]
            t = [int(q) for q in rng.permutation(n)[:k]]
            s.apply_gate(t, u)
            want = oracle.apply_gate(want, n, u, t, [])
            count += 1 << k
        else:                    # a program: a few, tens, hundreds of KiB
            depth = (1, 8, 60)[k] if rng.random() < 0.5 else 1
            gates = layered_circuit(n, depth, int(rng.integers(1 << 30)))
            s.apply_fused(qsv.Circuit.from_gates(gates))
            want = oracle.simulate(n, gates, init=want)
            count += len(gates)
    got = s.get()
    s.free()
    # a rounding of an amplitude (at most 1) per gate of one target, and per
    # term of a row of a larger one, adding up like a random walk or better
    eps = 2.0 ** -24 if prec == C64 else 2.0 ** -53
    assert np.max(np.abs(got - want)) <= 8 * eps * np.sqrt(count)

"""Diagonal gates of one to five targets under controls on every kind of qubit:
below a cache line, at one, above, and several, on states from fewer
amplitudes than a work-group has threads up.

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
@pytest.mark.parametrize("n", [5, 7, 8, 9, 11, 12, 19])
def test_tables_under_controls(n, prec):
    rng = np.random.default_rng(n)
    s = qsv.State(n, prec)
    psi = random_state(n, n)
    if prec == qsv.QSV_C64:
        psi = psi.astype(np.complex64).astype(np.complex128)
    for controls in ([2], [3], [2, 3], [3, 4], [3, n - 1], [0, 3], [8],
                     [8, n - 1]):
        if max(controls) >= n or len(set(controls)) < len(controls):
            continue
        free = [q for q in range(n) if q not in controls]
        for k in (1, 2, 3, 5):
            if len(free) < k:
                continue
            for t in (free[:k], free[-k:],
                      [int(q) for q in rng.permutation(free)[:k]]):
                d = np.exp(1j * rng.uniform(0, 6.28, 1 << k))
                s.set(psi)
                s.apply_gate(t, np.diag(d), controls)
                want = oracle.apply_gate(psi, n, np.diag(d), t, controls)
                err = np.max(np.abs(s.get() - want))
                assert err <= 4 * EPS[prec], (k, controls, t, err)
    s.free()


# From 2^29 amplitudes up other forms are chosen, and a grid may take several
# rounds over them.
@pytest.mark.parametrize("prec", [qsv.QSV_C64, qsv.QSV_C128])
@pytest.mark.parametrize("targets,control", [([7], 3), ([7, 15], 3),
                                             ([0, 7, 15], 3), ([7], None),
                                             ([4], 15)])
def test_tables_and_phases_of_large_states(targets, control, prec):
    n = 30
    dtype = torch.complex64 if prec == qsv.QSV_C64 else torch.complex128
    rng = np.random.default_rng(n)
    row = rng.uniform(-.7, .7, 1 << 16) + 1j * rng.uniform(-.7, .7, 1 << 16)
    row = torch.tensor(row, dtype=dtype, device="cuda")
    psi = row.repeat(1 << (n - 16))
    d = np.exp(1j * rng.uniform(0, 6.28, 1 << len(targets)))
    if targets == [4]:
        d[0] = 1                 # a phase where the target is 1
    want = oracle.apply_gate(row.cpu().numpy().astype(np.complex128), 16,
                             np.diag(d), targets,
                             [] if control is None else [control])
    want = torch.tensor(want, device="cuda")
    torch.cuda.synchronize()
    s = qsv.State(n, prec, tensor=psi)
    s.apply_gate(targets, np.diag(d), [] if control is None else [control])
    s.sync()
    err = max(float((p - want).abs().max())
              for p in psi.view(-1, 1 << 8, 1 << 16))
    assert err <= 4 * EPS[prec], err
    s.free()
    del psi
    torch.cuda.empty_cache()

"""What a call may take: device memory only where it needs some."""
import numpy as np
import pytest

import oracle
from circuits import layered_circuit

torch = pytest.importorskip("torch")
from paper_2502_11385_amd import qsv  # noqa: E402

pytestmark = pytest.mark.gpu
C64, C128 = qsv.QSV_C64, qsv.QSV_C128


@pytest.fixture(autouse=True)
def _need_gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    yield
    qsv.debug_inject(1, 0)


@pytest.mark.parametrize("prec", [C64, C128])
def test_plan_without_a_program_allocates_nothing(prec):
    """Gates of one and two targets run from kernel arguments, an empty
    circuit not at all: no program buffer."""
    n, gates = 9, layered_circuit(9, 3, 2)
    plain = qsv.fuse_opts(strategy=qsv.PLAN_PLAIN)
    s = qsv.State(n, prec)
    s.init_basis(5)
    qsv.debug_inject(1, 1)
    s.apply_fused(qsv.Circuit())
    s.apply_fused(qsv.Circuit.from_gates(gates), plain)
    got = s.get()
    want = oracle.simulate(n, gates, init=5)
    tol = (2.0 ** -22 if prec == C64 else 2.0 ** -50) * len(gates)
    assert np.max(np.abs(got - want)) <= tol
    s.free()


@pytest.mark.parametrize("prec", [C64, C128])
def test_folded_probabilities_allocate_nothing(prec):
    """The last tile pass writes the probabilities itself: no scratch."""
    n, gates = 14, layered_circuit(14, 6, 3)
    circ = qsv.Circuit.from_gates(gates)
    s = qsv.State(n, prec)
    out = torch.empty(1 << n, dtype=torch.float64, device="cuda")
    s.init_basis(0)
    s.apply_fused(circ)          # takes the program buffer
    s.init_basis(0)
    qsv.debug_inject(1, 1)
    s.apply_fused_outputs(circ, probs_ptr=out.data_ptr(), probs_fp64=True)
    assert s.plan_stats()["folded_outputs"] == 1
    s.sync()
    got = out.cpu().numpy()
    want = oracle.probabilities(oracle.simulate(n, gates))
    # an amplitude's error as above, twice its modulus (at most 1) in p
    tol = (2.0 ** -21 if prec == C64 else 2.0 ** -49) * len(gates)
    assert np.max(np.abs(got - want)) <= tol
    s.free()

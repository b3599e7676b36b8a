"""Passes launched while later ones are being planned: a state's first call
sizes its buffers and launches the circuit whole, later calls may launch it
in parts.  Both give the oracle's state and the same bits."""
import numpy as np
import pytest

import oracle
from circuits import layered_circuit, qft_style_circuit

torch = pytest.importorskip("torch")
from paper_2502_11385_amd import qsv  # noqa: E402

pytestmark = pytest.mark.gpu
C64, C128 = qsv.QSV_C64, qsv.QSV_C128


@pytest.fixture(scope="module", autouse=True)
def _need_gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


# (qubits, gates): one pass; the fewest gates that can be split; many passes;
# a program beyond the early bound (never split)
def _circuit(name):
    if name == "one":
        return 12, 0, layered_circuit(12, 8, 5)
    if name == "few":
        return 14, 0, layered_circuit(14, 10, 6)
    if name == "qft":
        x, g = qft_style_circuit(16, 9, tail_layers=4)
        return 16, x, g
    if name == "many":
        return 16, 0, layered_circuit(16, 60, 7)
    return 13, 0, layered_circuit(13, 110, 8)


@pytest.mark.parametrize("prec", [C64, C128])
@pytest.mark.parametrize("name", ["one", "few", "qft", "many", "large"])
def test_repeated_calls_give_the_same_state(name, prec):
    n, x, gates = _circuit(name)
    if name == "large":
        assert len(gates) * 1024 > 2 << 20
    want = oracle.simulate(n, gates, init=x)
    circ = qsv.Circuit.from_gates(gates)
    qs = [0, n // 2, n - 1]
    s = qsv.State(n, prec)
    runs, stats = [], []
    for i in range(4):
        s.init_basis(x)
        s.sync()                 # the stream is idle when the call begins
        if i % 2:
            s.apply_fused(circ)
            marg = s.marginal(qs)
        else:
            marg, shots = s.apply_fused_outputs(circ, marg_qubits=qs,
                                                shots=64, seed=3)
        st = s.plan_stats()
        stats.append({k: st[k] for k in ("passes", "gates", "segments")})
        runs.append((s.get(), marg))
    # rounding: every gate adds at most about one unit in the last place
    eps = 2.0 ** -24 if prec == C64 else 2.0 ** -53
    tol = 4 * eps * np.sqrt(len(gates)) + 1e-14
    mtol = 2e-6 if prec == C64 else 1e-12
    for amps, marg in runs:
        assert np.array_equal(amps, runs[0][0])
        assert np.max(np.abs(amps - want)) <= tol
        p = np.abs(amps.astype(complex)) ** 2
        assert np.max(np.abs(marg - oracle.marginal(p, n, qs))) <= mtol
    assert all(t == stats[0] for t in stats)
    s.free()


@pytest.mark.parametrize("prec", [C64, C128])
def test_allocation_failure_keeps_the_state(prec):
    """A call whose buffers have to grow (here: the shots' scratch) is
    launched whole or not at all."""
    n, _, gates = _circuit("few")
    longer = layered_circuit(14, 60, 6)
    s = qsv.State(n, prec)
    s.init_basis(0)
    s.apply_fused(qsv.Circuit.from_gates(gates))
    s.apply_fused(qsv.Circuit.from_gates(gates))
    before = s.get()
    qsv.debug_inject(1, 1)
    try:
        with pytest.raises(qsv.QsvError) as e:
            s.apply_fused_outputs(qsv.Circuit.from_gates(longer), shots=64)
        assert e.value.status == qsv.QSV_ERR_OUT_OF_MEMORY
    finally:
        qsv.debug_inject(1, 0)
    assert np.array_equal(s.get(), before)
    s.apply_fused(qsv.Circuit.from_gates(longer))
    want = oracle.simulate(n, gates + gates + longer)
    eps = 2.0 ** -24 if prec == C64 else 2.0 ** -53
    tol = 4 * eps * np.sqrt(len(gates) * 2 + len(longer)) + 1e-14
    assert np.max(np.abs(s.get() - want)) <= tol
    s.free()

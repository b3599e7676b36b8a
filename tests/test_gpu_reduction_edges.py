"""Reductions at the sizes where their split changes: the norm and Pauli sums
around one block, one block per chunk and the cap on the blocks, with more
terms than one launch takes.

Tolerances: a compensated FP64 sum of 2^n terms of a normalised state is off
by a few units in the last place of 1; 1e-13 allows for the products' own
rounding (2^n terms of size 2^-n, each off by at most 2^-52 of itself).
"""
import numpy as np
import pytest

import oracle
from circuits import random_state

torch = pytest.importorskip("torch")
from paper_2502_11385_amd import qsv  # noqa: E402

pytestmark = pytest.mark.gpu

C64, C128 = qsv.QSV_C64, qsv.QSV_C128
DT = {C64: np.complex64, C128: np.complex128}


@pytest.fixture(scope="module", autouse=True)
def _need_gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


def _state(psi, prec):
    s = qsv.State(int(np.log2(psi.size)), prec)
    s.set(psi)
    return s


@pytest.mark.parametrize("prec", [C64, C128])
@pytest.mark.parametrize("n", [1, 2, 8, 9, 10, 19, 20, 21])
def test_norm_and_pauli_edges(n, prec):
    psi = random_state(n, 40 + n).astype(DT[prec])
    rng = np.random.default_rng(n)
    terms = [{q: "XYZ"[int(rng.integers(3))] for q in range(n)
              if rng.random() < 0.5} for _ in range(5)]
    terms += [{}, {n - 1: "Z"}, {0: "X"}, {n - 1: "Y"}]
    s = _state(psi, prec)
    got = s.expectation(terms)
    norm = s.norm()
    s.free()
    wide = psi.astype(np.complex128)
    want = [oracle.pauli_expectation(wide, n, t) for t in terms]
    assert np.max(np.abs(got - want)) <= 1e-13
    assert abs(norm - oracle.norm(wide)) <= 1e-13


def test_more_pauli_terms_than_one_launch():
    n = 7
    psi = random_state(n, 3)
    rng = np.random.default_rng(5)
    terms = [{int(q): "XYZ"[int(rng.integers(3))]
              for q in rng.permutation(n)[:int(rng.integers(0, n + 1))]}
             for _ in range(130)]
    s = _state(psi, C128)
    got = s.expectation(terms)
    s.free()
    want = [oracle.pauli_expectation(psi, n, t) for t in terms]
    assert np.max(np.abs(got - want)) <= 1e-13


@pytest.mark.parametrize("prec", [C64, C128])
@pytest.mark.parametrize("n,k", [(1, 2), (13, 1), (13, 8192), (14, 100),
                                 (16, 1), (16, 100), (16, 30000)])
def test_top_k_gather_and_refine(n, k, prec):
    """A state with few distinct magnitudes, so that from 16 qubits the k-th
    key's bin holds more keys than the gather has room for and the digits
    decide; below, and for k near 2^n, the gather does."""
    rng = np.random.default_rng(n + k)
    psi = (rng.integers(1, 4, 1 << n) *
           np.exp(1j * rng.integers(0, 4, 1 << n) * np.pi / 2)).astype(DT[prec])
    s = _state(psi, prec)
    idx, p = s.top_k(k)
    s.free()
    widx, wp = oracle.top_k(oracle.probs_of_amplitudes(psi), k)
    assert idx.tolist() == widx.tolist()
    assert p.tolist() == wp.tolist()


@pytest.mark.parametrize("n", [1, 10, 11, 16, 17, 20])
def test_sample_block_search_edges(n):
    """1, 2, 64, 128 and 1024 blocks; all weight on one amplitude of the first
    or the last block, then spread out: the least index with C(i) > t, where
    no step of the cumulative sum lies within 1e-9 of t."""
    shots = 2000
    for where in (0, (1 << n) - 1):
        psi = np.zeros(1 << n, np.complex128)
        psi[where] = 1
        s = _state(psi, C128)
        assert np.all(s.sample(shots, 11) == where)
        s.free()
    psi = random_state(n, n)
    s = _state(psi, C128)
    got = s.sample(shots, 12)
    s.free()
    p = oracle.probabilities(psi)
    c = np.cumsum(p)
    t = oracle.uniforms(12, shots) * c[-1]
    want = np.searchsorted(c, t, side="right")
    off = np.nonzero(got != want)[0]
    for j in off:
        lo, hi = sorted((int(got[j]), int(want[j])))
        assert np.min(np.abs(c[lo:hi] - t[j])) <= 1e-9

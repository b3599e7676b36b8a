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

"""Relabelling at the edges of its tiles: states of fewer qubits than a tile
spans, permutations that keep, swap or scatter the lowest qubits, wrapped and
owned states, and states larger than the last-level cache.  The moved
amplitudes are the same bits."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
from paper_2502_11385_amd import qsv  # noqa: E402

pytestmark = pytest.mark.gpu

C64, C128 = qsv.QSV_C64, qsv.QSV_C128
CT = {C64: torch.complex64, C128: torch.complex128}


@pytest.fixture(scope="module", autouse=True)
def _need_gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


def _perms(n, rng):
    yield list(range(n))[::-1]
    yield list(range(1, n)) + [0]
    yield [1, 0] + list(range(2, n))                   # low swap only
    yield list(range(n - 2)) + [n - 1, n - 2]          # high swap only
    yield [int(q) for q in rng.permutation(n)]


def _moved(t, perm):
    n = len(perm)
    at = torch.arange(1 << n, device=t.device)
    src = torch.zeros_like(at)
    for q, to in enumerate(perm):
        src |= (at >> to & 1) << q
    return t[src]


@pytest.mark.parametrize("prec", [C64, C128])
@pytest.mark.parametrize("n", [2, 3, 5, 8, 9, 11, 12, 13, 14, 18])
def test_small_states(n, prec):
    rng = np.random.default_rng(n)
    for perm in _perms(n, rng):
        t = torch.randn(1 << n, dtype=CT[prec], device="cuda")
        want = _moved(t, perm)
        s = qsv.State(n, prec)
        s.set(t.cpu().numpy())
        s.permute_qubits(perm)
        assert np.array_equal(s.get(), want.cpu().numpy()), perm
        s.free()
        w = qsv.State(n, prec, tensor=t)
        w.permute_qubits(perm)
        w.sync()
        assert torch.equal(t, want), perm
        w.free()


@pytest.mark.parametrize("n,prec", [(26, C64), (25, C128)])
def test_larger_than_the_cache(n, prec):
    rng = np.random.default_rng(n)
    perm = [int(q) for q in rng.permutation(n)]
    t = torch.randn(1 << n, dtype=CT[prec], device="cuda")
    want = _moved(t, perm)
    w = qsv.State(n, prec, tensor=t)
    w.permute_qubits(perm)
    w.sync()
    assert torch.equal(t, want)
    w.free()

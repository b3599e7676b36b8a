"""Top-k where 2^32 or more keys are equal, so that 32 bits cannot count them:
the selection is the first k indices, exactly."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
from paper_2502_11385_amd import qsv  # noqa: E402

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _need_gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


# (qubits, equal amplitudes, k); the others are 0.  With 2^32 + 16 equal keys
# a 32-bit count reads 16, which would pass for a bin that fits.
@pytest.mark.parametrize("n,equal,k", [(32, 1 << 32, 8), (33, 1 << 32, 8),
                                       (33, (1 << 32) + 16, 8),
                                       (33, 1 << 33, 65536)])
def test_top_k_of_more_equal_keys_than_32_bits_count(n, equal, k):
    v = 2.0 ** -16
    psi = torch.zeros(1 << n, dtype=torch.complex64, device="cuda")
    psi[:equal] = v
    torch.cuda.synchronize()
    s = qsv.State(n, qsv.QSV_C64, tensor=psi)
    for _ in range(2):           # on new scratch, and on the first call's
        idx, p = s.top_k(k)
        assert np.array_equal(idx, np.arange(k, dtype=np.uint64))
        assert np.all(p == v * v)
    s.free()
    del psi
    torch.cuda.empty_cache()

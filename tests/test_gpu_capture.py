"""Calls on a stream under capture: those that only launch kernels replay as
they ran, those that upload a program are refused, as a replay would read
buffers that later calls overwrite and free."""
import numpy as np
import pytest

from circuits import layered_circuit, random_state

torch = pytest.importorskip("torch")
from paper_2502_11385_amd import qsv  # noqa: E402

pytestmark = pytest.mark.gpu
C64, C128 = qsv.QSV_C64, qsv.QSV_C128
N = 13
U = np.linalg.qr(random_state(4, 1).reshape(4, 4))[0]
M = np.linalg.qr(random_state(6, 2).reshape(8, 8))[0]
GATES = layered_circuit(N, 4, 9)


@pytest.fixture(scope="module", autouse=True)
def _need_gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


def _capture(stream, call):
    g = torch.cuda.CUDAGraph()
    with torch.cuda.stream(stream):
        g.capture_begin(capture_error_mode="relaxed")
        try:
            call()
        finally:
            g.capture_end()
    return g


LAUNCHES = {
    "gate": lambda s, out: s.apply_gate([2, 9], U, controls=[5]),
    "diagonal": lambda s, out: s.apply_gate([7], np.diag([1, 1j])),
    "plain": lambda s, out: s.apply_fused(
        qsv.Circuit.from_gates(GATES), qsv.fuse_opts(strategy=qsv.PLAN_PLAIN)),
    "probabilities": lambda s, out: s.probabilities_into(out.data_ptr(), True),
}


@pytest.mark.parametrize("prec", [C64, C128])
@pytest.mark.parametrize("name", sorted(LAUNCHES))
def test_launches_replay(name, prec):
    call = LAUNCHES[name]
    psi = random_state(N, 4)
    st = torch.cuda.Stream()
    out = torch.zeros(1 << N, dtype=torch.float64, device="cuda")
    torch.cuda.synchronize()
    s = qsv.State(N, prec, stream=st)
    s.set(psi)
    call(s, out)
    s.sync()
    want, pwant = s.get(), out.cpu().numpy()
    g = _capture(st, lambda: call(s, out))
    for i in range(3):
        s.set(psi)
        out.zero_()
        torch.cuda.synchronize()
        with torch.cuda.stream(st):
            g.replay()
        torch.cuda.synchronize()
        assert np.array_equal(s.get(), want)
        assert np.array_equal(out.cpu().numpy(), pwant)
        s.apply_fused(qsv.Circuit.from_gates(GATES))   # eager work between
        s.norm()
    s.free()


UPLOADS = {
    "tiled": lambda s: s.apply_fused(qsv.Circuit.from_gates(GATES)),
    "fused": lambda s: s.apply_fused(
        qsv.Circuit.from_gates(GATES), qsv.fuse_opts(strategy=qsv.PLAN_FUSED)),
    "matrix": lambda s: s.apply_gate([1, 5, 9], M),
    "block": lambda s: s.apply_gate([1, 3, 5, 9], np.kron(U, U)),
}


@pytest.mark.parametrize("prec", [C64, C128])
@pytest.mark.parametrize("name", sorted(UPLOADS))
def test_program_uploads_are_refused(name, prec):
    call = UPLOADS[name]
    st = torch.cuda.Stream()
    s, other = qsv.State(N, prec, stream=st), qsv.State(N, prec)
    s.init_basis(0)
    call(s)                      # the buffers are there
    s.sync()
    errors = []

    def captured():
        s.init_basis(0)
        try:
            call(s)
        except qsv.QsvError as e:
            errors.append(e.status)

    _capture(st, captured)
    assert errors == [qsv.QSV_ERR_DEVICE]
    other.init_basis(0)
    call(other)                  # other states are unaffected
    assert abs(other.norm() - 1) < 1e-5
    other.free()
    s.free()

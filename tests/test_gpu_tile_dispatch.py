"""Tile passes on scattered qubits: the runs of outer qubits that place a
tile (one, four, and more than four), every register width's re-layouts, and
multi-controlled ops whose controls lie all inside the tile, all outside it,
or on both sides.

Tolerances: 1e-12 (complex128) and 1e-6 (complex64) absolute per amplitude.
"""
import numpy as np
import pytest

import oracle
from circuits import batch_variants, random_state

torch = pytest.importorskip("torch")
from paper_2502_11385_amd import qsv  # noqa: E402

pytestmark = pytest.mark.gpu

C64, C128 = qsv.QSV_C64, qsv.QSV_C128
TOL = {C64: 1e-6, C128: 1e-12}

# tile qubits (8 of 16, qubit 0 always) and the runs of outer qubits they leave
TILES = {1: (1, 2, 3, 4, 5, 6, 7), 4: (2, 3, 5, 7, 8, 10, 11),
         6: (1, 4, 6, 8, 10, 13, 15)}


@pytest.fixture(scope="module", autouse=True)
def _need_gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


def _unitary(rng):
    z = rng.standard_normal((2, 2)) + 1j * rng.standard_normal((2, 2))
    q, r = np.linalg.qr(z)
    return q * (np.diag(r) / np.abs(np.diag(r)))


@pytest.mark.parametrize("prec,reg", [(C64, 3), (C64, 4), (C64, 5),
                                      (C128, 3), (C128, 4)])
@pytest.mark.parametrize("runs", sorted(TILES))
def test_scattered_tile(runs, prec, reg):
    n, tile = 16, TILES[runs]
    outer = [q for q in range(1, n) if q not in tile]
    rng = np.random.default_rng(100 * runs + reg)
    gates = [((q,), _unitary(rng), ()) for q in tile]
    for i in range(24):
        t, a, b = rng.permutation(tile)[:3]
        x, y = rng.permutation(outer)[:2]
        controls = ((a,), (x,), (a, b), (x, y), (a, x), ())[i % 6]
        gates.append(((t,), _unitary(rng), tuple(int(c) for c in controls)))
    circ = qsv.Circuit()
    want = random_state(n, runs)
    s = qsv.State(n, prec)
    s.set(want)
    for t, u, c in gates:
        circ.add([int(q) for q in t], u, c)
        want = oracle.apply_gate(want, n, u, [int(q) for q in t], list(c))
    s.apply_fused(circ, qsv.fuse_opts(strategy=qsv.PLAN_TILED, tile_log2=8,
                                      low_qubits=1, reg_log2=reg))
    got = s.get().astype(np.complex128)
    s.free()
    assert np.max(np.abs(got - want)) <= TOL[prec]


# state sizes on both sides of the line between whole and half re-layouts
# (32 MiB), and a tile too large to go whole in a small state
@pytest.mark.parametrize("prec,n,tile", [(C64, 22, 12), (C64, 23, 12),
                                         (C64, 16, 13),
                                         (C128, 21, 12), (C128, 22, 12),
                                         (C128, 15, 13)])
def test_whole_and_half_relayouts(prec, n, tile):
    rng = np.random.default_rng(n + tile)
    qs = sorted({int(q) for q in rng.permutation(n)[:9]} | {0, n - 1})
    circ = qsv.Circuit()
    want = random_state(n, 3)
    s = qsv.State(n, prec)
    s.set(want)
    for i in range(3):
        for j, q in enumerate(qs):
            u = _unitary(rng)
            c = [qs[j - 1]] if i == 1 and j else []
            circ.add([q], u, c)
            want = oracle.apply_gate(want, n, u, [q], c)
    s.apply_fused(circ, qsv.fuse_opts(strategy=qsv.PLAN_TILED, tile_log2=tile,
                                      reg_log2=4))
    assert np.max(np.abs(s.get() - want)) <= TOL[prec]
    s.free()


def test_batches_on_both_sides_of_the_relayout_line():
    """The same variants in a batch of few tiles (whole re-layouts) and of
    more than 2048 (halves, complex64): the oracle's vectors, the same bits."""
    vs = batch_variants(count=2, seed=5, wmin=18, wmax=18, dmin=3, dmax=4)
    got = []
    for copies in (1, 20):
        b = qsv.Batch(vs * copies, prec=C64)
        out = b.output()
        b.launch(out)
        torch.cuda.synchronize()
        got.append(out.cpu().numpy())
        assert (int(b.offsets[-1]) >> 12 > 2048) == (copies == 20)
        b.free()
    size = got[0].size
    for c in range(20):
        assert np.array_equal(got[1][c * size:(c + 1) * size], got[0]), c
    for i, v in enumerate(vs):
        want = oracle.variant_probabilities(v)
        p = got[0][i << 18:(i + 1) << 18].astype(np.float64)
        assert np.max(np.abs(p - want)) <= 2e-6

"""Cut reconstruction above eight uncut qubits, where a work-group takes rows
of 256 outcomes: every split of the subcircuits into varying and uniform ones
and of the qubits into rows, with the outputs in order and scattered, and the
chain whose varying subcircuits touch too many cuts for it.

Tolerance: the sums have up to 64 products of entries of size 1; each product
and sum is off by at most a few 2^-53, relative to the largest result.
"""
import numpy as np
import pytest

import oracle
from circuits import cut_chain, cut_variants

torch = pytest.importorskip("torch")
from paper_2502_11385_amd import qsv  # noqa: E402

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _need_gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


@pytest.mark.parametrize("scatter", [False, True])
@pytest.mark.parametrize("widths", [(9,), (9, 2), (3, 8), (9, 4, 3), (4, 4, 8),
                                    (10, 3, 4), (8, 8), (2, 2, 2, 8),
                                    (9, 3, 2, 3)])
def test_rows_and_splits(widths, scatter):
    prob = cut_chain(widths, 1, 7)
    rng = np.random.default_rng(sum(widths))
    if scatter:
        to = rng.permutation(prob.n)
        for sub in prob.subs:
            sub.out_qubit = [int(to[q]) if q >= 0 else -1
                             for q in sub.out_qubit]
    vp = [[rng.standard_normal(1 << sub.width) for _ in cut_variants(sub)]
          for sub in prob.subs]
    flat = np.concatenate([v for vs in vp for v in vs])
    lens = [len(v) for vs in vp for v in vs]
    offs = np.concatenate([[0], np.cumsum(lens)[:-1]]).astype(np.uint64)
    out = torch.full((1 << prob.n,), float("nan"), dtype=torch.float64,
                     device="cuda")
    qsv.cut_reconstruct(qsv.CutSpec(prob.n, prob.n_cuts, prob.subs),
                        torch.from_numpy(flat).cuda(), offs, out)
    got = out.cpu().numpy()
    want = oracle.cut_reconstruct(prob, vp)
    assert np.max(np.abs(got - want)) <= 1e-13 * np.max(np.abs(want))

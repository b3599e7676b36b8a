"""Cut reconstruction where a work-group's sums over the uniform subcircuits'
term choices are split over its threads: fewer sums than threads, from one
round to many, and more rows per work-group.

Tolerance: up to 4^5 products, each off by a few 2^-53 of itself, added one
after the other: 1040 * 2^-53 of the sum of their moduli, which for random
signs is about 32 of a result's usual size, 8 of the largest's: 1e-12 of it.
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


@pytest.mark.parametrize("widths", [(9, 2, 4, 3), (9, 2, 2, 2, 2),
                                    (9, 2, 2, 2, 2, 2), (5, 5, 2, 2, 2),
                                    (9, 1, 2, 1, 2), (9, 4, 4, 7)])
def test_sums_over_many_term_choices(widths):
    prob = cut_chain(widths, 1, 7)
    rng = np.random.default_rng(sum(widths))
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
    assert np.max(np.abs(got - want)) <= 1e-12 * np.max(np.abs(want))

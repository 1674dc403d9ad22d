"""Batches of many graphs much smaller than a block of the statistics' sums
holds, and of as many that mean sizes fall on either side of its sizes.
Whole numbers throughout: every result must equal the oracle's."""

import numpy as np
import pytest

import oracle
from paper_1610_08128_amd import inputs as I

pytestmark = pytest.mark.gpu


def _some(rng, n):
    u, v = rng.integers(0, n, 2 * n), rng.integers(0, n, 2 * n)
    keep = u != v
    return I.from_edges(n, u[keep], v[keep])


@pytest.mark.parametrize("count,lo,hi", [(2000, 1, 1), (1500, 1, 4), (700, 10, 23), (300, 15, 18),
                                         (60, 300, 700), (40, 511, 514), (5, 8000, 9000),
                                         (3, 16383, 16385), (2, 1, 40000)])
def test_batches(count, lo, hi):
    import torch
    from paper_1610_08128_amd import rcm

    rng = np.random.default_rng(count)
    graphs = [_some(rng, int(n)) for n in rng.integers(lo, hi + 1, count)]
    vo, no, rp, ci = I.concat_batch(graphs)
    print(f"{count} graphs of {lo} to {hi}: {int(vo[-1])} vertices", flush=True)
    perm, stats = rcm.order_batched(vo, no, torch.from_numpy(rp).cuda(),
                                    torch.from_numpy(ci).cuda())
    perm = perm.cpu().numpy()
    for i, g in enumerate(graphs):
        want = oracle.rcm(g.n, g.rowptr, g.colidx)
        assert np.array_equal(perm[vo[i]:vo[i + 1]], want.perm), i
        assert stats[i] == want.stats, i

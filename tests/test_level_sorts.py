"""The level orders' sorts: position key and degree in one key (bounded rows,
small graphs) and one after the other (long rows in larger graphs), on either
side of the sizes at which the number of passes changes.  Whole numbers
throughout: every result must equal the oracle's."""

import numpy as np
import pytest

import oracle
from paper_1610_08128_amd import inputs as I

pytestmark = pytest.mark.gpu


def _graphs(n):
    rng = np.random.default_rng(n)
    i = np.arange(n)
    # rows of up to 8, and one long row with the same edges besides
    u, v = np.concatenate([i, i]), np.concatenate([(i + 1) % n, rng.permutation(n)])
    keep = u != v
    yield I.from_edges(n, u[keep], v[keep], name=f"bounded_{n}")
    w = rng.integers(1, n, min(n, 300))
    yield I.from_edges(n, np.concatenate([u[keep], np.zeros(w.size, np.int64)]),
                       np.concatenate([v[keep], w]), name=f"hub_{n}")


@pytest.mark.parametrize("n", [2, 15, 16, 17, 255, 257, 2048, 4095, 4097, 65535, 65537, 70000])
@pytest.mark.parametrize("label_mode", [1, 2])
def test_orders(n, label_mode):
    import torch
    from paper_1610_08128_amd import rcm

    for g in _graphs(n):
        want = oracle.rcm(g.n, g.rowptr, g.colidx, cm_mode=label_mode + 1)
        assert want.status == oracle.OK
        perm, iperm, st = rcm.order(torch.from_numpy(g.rowptr).cuda(),
                                    torch.from_numpy(g.colidx).cuda(), return_iperm=True,
                                    label_mode=label_mode)
        assert np.array_equal(perm.cpu().numpy(), want.perm), g.name
        assert np.array_equal(iperm.cpu().numpy(), want.iperm), g.name
        assert st == want.stats, g.name

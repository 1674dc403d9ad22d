"""The team kernel's parents on rows longer than a register batch, with as many
children as are ranked in registers at once, one more and fewer, on both
work-group sizes.  Whole numbers throughout: every result must equal the
oracle's."""

import numpy as np
import pytest

import oracle
from paper_1610_08128_amd import inputs as I

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("threads", [256, 512])
@pytest.mark.parametrize("kids", [7, 8, 9, 11, 12, 13, 25])
def test_children_per_long_row(threads, kids):
    """A path of 300 vertices with 0 to kids - 1 leaves on each, so a row of
    up to kids + 2 entries has up to kids children at its parent's level."""
    import torch
    from paper_1610_08128_amd import rcm

    rng = np.random.default_rng(kids)
    leaves = rng.integers(0, kids, 300)
    leaves[::7] = kids - 1
    owner = np.repeat(np.arange(300), leaves)
    n = 300 + owner.size
    u = np.concatenate([np.arange(299), owner])
    v = np.concatenate([np.arange(1, 300), np.arange(300, n)])
    label = rng.permutation(n)
    g = I.from_edges(n, label[u], label[v], name=f"leaves_{kids}")
    want = oracle.rcm(g.n, g.rowptr, g.colidx)
    rp, ci = torch.from_numpy(g.rowptr).cuda(), torch.from_numpy(g.colidx).cuda()
    for opts in ({"team_size": 1}, {"team_size": 4, "narrow_cutoff": -1}):
        perm, iperm, st = rcm.order(rp, ci, return_iperm=True, mode=1, block_threads=threads,
                                    small_cutoff=1, **opts)
        assert np.array_equal(perm.cpu().numpy(), want.perm), opts
        assert np.array_equal(iperm.cpu().numpy(), want.iperm), opts
        assert st == want.stats

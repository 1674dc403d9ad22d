"""The row checks of graphs with long rows, 16 lanes a row: repeated columns at
every distance, rows of the lengths at which a lane's second entry, the
re-reading of the row or the check by hashing begins, ascending or not, bad
columns and bounds, and the rows' copy for those that fit it.  The team path
(mode 1); every result must equal the oracle's."""

import numpy as np
import pytest

import oracle
from paper_1610_08128_amd import inputs as I

pytestmark = pytest.mark.gpu


def _status(rp, ci, **opts):
    import torch
    from paper_1610_08128_amd import rcm

    try:
        rcm.order(torch.from_numpy(np.asarray(rp, np.int32)).cuda(),
                  torch.from_numpy(np.asarray(ci, np.int32)).cuda(), mode=1, **opts)
    except rcm.RcmError as e:
        return e.status
    return rcm.OK


def _rows(g):
    return [g.colidx[g.rowptr[i]:g.rowptr[i + 1]].copy() for i in range(g.n)]


@pytest.mark.parametrize("length", [9, 15, 16, 17, 31, 32, 33, 48, 63, 64, 65, 100])
def test_repeated_columns(length):
    from paper_1610_08128_amd import rcm

    # (complete rows of that length: every vertex of length - 1 others)
    g = I.disjoint_union([I.complete(length)] * 3, seed=length)
    rng = np.random.default_rng(length)
    rows = _rows(g)
    assert _status(g.rowptr, np.concatenate(rows)) == rcm.OK
    shuffled = [rng.permutation(r) for r in rows]
    assert _status(g.rowptr, np.concatenate(shuffled)) == rcm.OK
    for at in range(0, length, 1 if length < 40 else 5):
        for base in (rows, shuffled):
            bad = [r.copy() for r in base]
            row = int(rng.integers(g.n))
            other = (at + 1 + int(rng.integers(length - 1))) % length
            bad[row][at] = bad[row][other]
            assert _status(g.rowptr, np.concatenate(bad)) == rcm.ERR_BAD_CSR, (row, at, other)
    for value in (-1, g.n, 2**31 - 1, -2**31):
        bad = [r.copy() for r in shuffled]
        bad[-1][-1] = value
        assert _status(g.rowptr, np.concatenate(bad)) == rcm.ERR_BAD_CSR
    for k, to in ((1, -1), (g.n // 2, 0), (g.n // 2, g.nnz + 1)):
        rp = g.rowptr.copy()
        rp[k] = to
        assert _status(rp, np.concatenate(rows)) == rcm.ERR_BAD_CSR


@pytest.mark.parametrize("n", [1, 15, 16, 63, 64, 65, 4097])
def test_results(n):
    """Rows of every length at once, ascending and not, with and without the
    diagonal, and empty ones: statistics and order."""
    import torch
    from paper_1610_08128_amd import rcm

    rng = np.random.default_rng(n)
    u = rng.integers(0, n, 9 * n)
    v = (rng.integers(0, n, 9 * n) * rng.random(9 * n) ** 2).astype(np.int64)
    keep = (u != v) & (u % 7 != 3) & (v % 7 != 3)
    g = I.from_edges(n, u[keep], v[keep], name=f"mixed_{n}")
    for h in (g, I.shuffle_rows(I.drop_diagonal(g), n)):
        if n > 1 and h.nnz <= 8 * n:
            continue
        want = oracle.rcm(h.n, h.rowptr, h.colidx)
        ci = h.colidx if h.colidx.size else np.zeros(1, np.int32)
        perm, iperm, st = rcm.order(torch.from_numpy(h.rowptr).cuda(),
                                    torch.from_numpy(ci).cuda(), return_iperm=True, mode=1)
        assert np.array_equal(perm.cpu().numpy(), want.perm)
        assert np.array_equal(iperm.cpu().numpy(), want.iperm)
        assert st == want.stats


def test_batch_segments():
    """A column of a neighbouring graph, in a long and in a short row."""
    import torch
    from paper_1610_08128_amd import rcm

    graphs = [I.complete(20), I.grid2d(30, 30, seed=1), I.complete(70), I.path(300, seed=2)]
    vo, no, rp, ci = I.concat_batch(graphs)
    args = [torch.from_numpy(rp).cuda()]

    def status(cols):
        try:
            rcm.order_batched(vo, no, args[0], torch.from_numpy(cols).cuda())
        except rcm.RcmError as e:
            return e.status
        return rcm.OK

    assert status(ci) == rcm.OK
    for i in range(len(graphs)):
        for k in (no[i], no[i + 1] - 1):
            bad = ci.copy()
            bad[k] = graphs[i].n
            assert status(bad) == rcm.ERR_BAD_CSR, (i, k)

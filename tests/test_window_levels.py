"""Levels of the window engine and of the bounded-row engine that one wave
walks without checks, at the widths that change how many lanes a vertex gets,
and components whose ids reach so far that the window's ends allow few such
levels or none.  Whole numbers throughout: every result must equal the
oracle's."""

import numpy as np
import pytest

import oracle
from paper_1610_08128_amd import inputs as I

pytestmark = pytest.mark.gpu


def _check(g, **opts):
    import torch
    from paper_1610_08128_amd import rcm

    print(f"case {g.name} n={g.n} nnz={g.nnz} {opts}", flush=True)
    want = oracle.rcm(g.n, g.rowptr, g.colidx, **opts)
    assert want.status == oracle.OK
    rp = torch.from_numpy(g.rowptr).cuda()
    ci = torch.from_numpy(g.colidx).cuda()
    perm, iperm, st = rcm.order(rp, ci, return_iperm=True, **opts)
    assert np.array_equal(perm.cpu().numpy(), want.perm), g.name
    assert np.array_equal(iperm.cpu().numpy(), want.iperm), g.name
    assert st == want.stats


@pytest.mark.parametrize("width", [1, 3, 7, 8, 9, 15, 16, 17, 31, 32, 33, 47, 64, 65])
def test_strip_widths(width):
    """The first structure starts inside the strip, so its levels are twice
    as wide as the later passes' (16, 32 and 64 vertices are the edges)."""
    for drop, seed in ((0.0, 1), (0.03, 2)):
        if width == 1 and drop:
            continue
        g = I.strip_drop(width, 9000, drop, seed) if width > 1 else I.path(12000, seed=3)
        _check(g)
        _check(g, pp_variant=1, reverse_mode=1)


@pytest.mark.parametrize("side", [8, 40, 70, 90])
def test_far_neighbours(side):
    """A square grid in the middle of a long path: levels up to `side` wide
    whose ids reach as far, with levels of one vertex around them."""
    tail = 6000
    i = np.arange(side * side).reshape(side, side)
    u = [i[:, :-1].ravel(), i[:-1].ravel()]
    v = [i[:, 1:].ravel(), i[1:].ravel()]
    n = side * side
    for corner in (0, side * side - 1):
        p = np.concatenate([[corner], n + np.arange(tail)])
        u.append(p[:-1])
        v.append(p[1:])
        n += tail
    g = I.from_edges(n, np.concatenate(u), np.concatenate(v),
                     perm=np.random.default_rng(side).permutation(n), name=f"grid_on_path_{side}")
    _check(g)


@pytest.mark.parametrize("width", [1, 2, 15, 16, 17, 31, 32, 33, 63, 64, 65])
def test_small_strip_widths(width):
    """Components in one work-group's LDS, with rows of at most 4 and of at
    most 8 off-diagonal entries, twice (the words of the first one are not
    free when the second is walked) and next to isolated vertices."""
    for diagonals in (False, True):
        m = min(2000 // width, 300)
        i = np.arange(width * m).reshape(m, width)
        u, v = [i[:, :-1].ravel(), i[:-1].ravel()], [i[:, 1:].ravel(), i[1:].ravel()]
        if diagonals:
            u += [i[:-1, :-1].ravel(), i[:-1, 1:].ravel()]
            v += [i[1:, 1:].ravel(), i[1:, :-1].ravel()]
        g = I.from_edges(i.size, np.concatenate(u), np.concatenate(v), name=f"strip_{width}")
        g = I.disjoint_union([g, I.path(1), g, I.path(1)], seed=width)
        for opts in ({}, {"pp_variant": 1, "reverse_mode": 1}, {"reverse_mode": 1}):
            _check(g, **opts)

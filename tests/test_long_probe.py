"""The first level structure of a long component of a graph past the component
engine's range, by one work-group: what it measures, declines and leaves to
the others.  Whole numbers throughout: every result must equal the oracle's."""

import numpy as np
import pytest

import oracle
from paper_1610_08128_amd import inputs as I

pytestmark = pytest.mark.gpu

RANGE = 1 << 19  # the engine's; the probe's ends at 1,146,880 vertices


def _strip(width, m, *, diagonals=False, tail=0):
    i = np.arange(width * m, dtype=np.int64).reshape(m, width)
    u, v = [i[:, :-1].ravel(), i[:-1].ravel()], [i[:, 1:].ravel(), i[1:].ravel()]
    if diagonals:
        u.append(i[:-1, :-1].ravel())
        v.append(i[1:, 1:].ravel())
    n = i.size
    if tail:
        # one row longer than the copy holds, at the strip's end
        u.append(np.full(tail, n - 1))
        v.append(n + np.arange(tail))
        n += tail
    return n, np.concatenate(u), np.concatenate(v)


def _graph(parts, seed, name, first=None):
    """Disjoint parts under random labels; vertex 0 in part `first`."""
    n, us, vs, starts = 0, [], [], []
    for k, u, v in parts:
        us.append(u + n)
        vs.append(v + n)
        starts.append(n)
        n += k
    perm = np.random.default_rng(seed).permutation(n)
    if first is not None:
        x = starts[first] + parts[first][0] // 2
        y = int(np.flatnonzero(perm == 0)[0])
        perm[x], perm[y] = perm[y], perm[x]
    return I.from_edges(n, np.concatenate(us), np.concatenate(vs), perm=perm, name=name)


def _cases():
    yield "strip_16", lambda: _graph([_strip(16, RANGE // 16 + 1)], 1, "strip_16"), 4
    yield "largest", lambda: _graph([_strip(20, 57344)], 2, "largest"), 4
    yield "past_largest", lambda: _graph([_strip(20, 57345)], 3, "past_largest"), 4
    yield "wide_levels", lambda: _graph([_strip(127, 4200)], 4, "wide_levels"), None
    yield "too_wide", lambda: _graph([_strip(130, 4100)], 5, "too_wide"), None
    yield "rows_of_6", lambda: _graph([_strip(24, 22000, diagonals=True)], 6, "rows_of_6"), 3
    yield "long_row", lambda: _graph([_strip(16, 33000, tail=20)], 7, "long_row"), None
    yield "head_and_rest", lambda: _graph([_strip(9, 30000), _strip(300, 1000), (1, *[np.zeros(0, np.int64)] * 2)], 8, "head_and_rest", first=0), 4
    yield "rows_of_6_and_rest", lambda: _graph([_strip(9, 30000, diagonals=True), _strip(300, 1000)], 9, "rows_of_6_and_rest", first=0), 3
    yield "small_head", lambda: _graph([_strip(30, 40), _strip(16, 33000)], 10, "small_head", first=0), None
    yield "isolated_head", lambda: _graph([(1, *[np.zeros(0, np.int64)] * 2), _strip(16, 33000)], 11, "isolated_head", first=0), None


CASES = list(_cases())


@pytest.mark.parametrize("idx", range(len(CASES)))
def test_long_components(idx):
    import torch
    from paper_1610_08128_amd import rcm

    name, make, mode = CASES[idx]
    g = make()
    print(f"case {name} n={g.n} nnz={g.nnz}", flush=True)
    rp = torch.from_numpy(g.rowptr).cuda()
    ci = torch.from_numpy(g.colidx).cuda()
    for opts in ({}, {"pp_variant": 1, "reverse_mode": 1}):
        want = oracle.rcm(g.n, g.rowptr, g.colidx, **opts)
        assert want.status == oracle.OK
        perm, iperm, st = rcm.order(rp, ci, return_iperm=True, **opts)
        if mode is not None and g.n <= 1146880:
            assert rcm.last_timings()["used_mode"] == mode
        assert np.array_equal(perm.cpu().numpy(), want.perm)
        assert np.array_equal(iperm.cpu().numpy(), want.iperm)
        assert st == want.stats

"""The 16-wave engine for small graphs with long rows at the sizes where it
can go wrong: rows at the lengths that change how they are checked and read
(16 and 32 entries), levels at the width where the ranking changes (256), the
sorts' and prefixes' shares (64, 1,024 vertices), isolated vertices, inputs it
must refuse.  Whole numbers throughout: every result must equal the oracle's."""

import numpy as np
import pytest

import oracle
from paper_1610_08128_amd import inputs as I

pytestmark = pytest.mark.gpu


def _check(g, **opts):
    import torch
    from paper_1610_08128_amd import rcm

    kw = {k: opts[k] for k in ("pp_variant", "reverse_mode") if k in opts}
    print(f"case {g.name} n={g.n} nnz={g.nnz} {opts}", flush=True)
    rp = torch.from_numpy(g.rowptr).cuda()
    ci = torch.from_numpy(g.colidx).cuda()
    perm, iperm, st = rcm.order(rp, ci, return_iperm=True, mode=2, **opts)
    assert rcm.last_timings()["used_block_threads"] == 1024, (g.name, g.n, g.nnz)
    want = oracle.rcm(g.n, g.rowptr, g.colidx, **kw)
    assert want.status == oracle.OK
    assert np.array_equal(perm.cpu().numpy(), want.perm), g.name
    assert np.array_equal(iperm.cpu().numpy(), want.iperm), g.name
    assert st == want.stats, (g.name, st, want.stats)


def _all_forms(g, seed):
    _check(g)
    _check(g, pp_variant=1, reverse_mode=1)
    _check(I.shuffle_rows(I.drop_diagonal(g), seed), check_full=True, reverse_mode=1)


def _relabelled(n, u, v, seed, name):
    return I.from_edges(n, np.asarray(u), np.asarray(v),
                        perm=np.random.default_rng(seed).permutation(n), name=name)


@pytest.mark.parametrize("length", [9, 15, 16, 17, 31, 32, 33, 64, 65, 100])
def test_row_lengths(length):
    """A ring whose vertices link to the next length / 2 ones, and a hub."""
    n = 4 * length + 300
    k = max(length // 2, 1)
    i = np.arange(n)
    u = np.concatenate([i for _ in range(k)] + [np.zeros(length, np.int64)])
    v = np.concatenate([(i + j + 1) % n for j in range(k)] +
                       [2 * length + np.arange(length)])
    _all_forms(_relabelled(n, u, v, length, f"ring_{length}"), length)


@pytest.mark.parametrize("width", [1, 63, 64, 65, 255, 256, 257, 1023, 1024, 1025])
def test_level_widths(width):
    """A root, a level of that width and one below it, their edges drawn at
    random: every child has several parents and the siblings many orders."""
    rng = np.random.default_rng(width)
    n = max(2 * width + 1, 300)
    a, b = 1 + np.arange(width), 1 + width + np.arange(width)
    u = np.concatenate([np.zeros(width, np.int64), b, b, rng.choice(a, width)])
    v = np.concatenate([a, rng.choice(a, width), rng.choice(a, width), rng.choice(b, width)])
    if width < 150:
        # (vertices left over: a ring of long rows)
        r = np.arange(2 * width + 1, n)
        u = np.concatenate([u] + [r for _ in range(5)])
        v = np.concatenate([v] + [np.roll(r, -j - 1) for j in range(5)])
    else:
        # (one long row at least, however the draws fell)
        u, v = np.concatenate([u, np.full(9, b[0])]), np.concatenate([v, a[:9]])
    _all_forms(_relabelled(n, u, v, width, f"levels_{width}"), width)


@pytest.mark.parametrize("n", [64, 65, 255, 256, 1023, 1024, 1025, 3000, 4000])
def test_sizes_and_isolated_vertices(n):
    """Random graphs of mean row 12 with every fifth vertex isolated."""
    rng = np.random.default_rng(n)
    live = np.flatnonzero(np.arange(n) % 5 != 3)
    u, v = rng.choice(live, 6 * live.size), rng.choice(live, 6 * live.size)
    keep = u != v
    u, v = u[keep], v[keep]
    if n < 256:
        # (mean row above 8 whatever is isolated)
        u, v = [x.ravel() for x in np.meshgrid(live, live)]
        u, v = u[u < v], v[u < v]
    _all_forms(_relabelled(n, u, v, n, f"isolated_{n}"), n)


@pytest.mark.parametrize("length", [10, 16, 17, 32, 33, 100])
def test_refused_inputs(length):
    """A column repeated at every distance within a row, a missing transpose
    entry under check_full, a column out of range."""
    import torch
    from paper_1610_08128_amd import rcm

    g = I.complete(max(length, 70))
    n = g.n
    rp = g.rowptr.astype(np.int32)
    rows = [g.colidx[rp[i]:rp[i + 1]].copy() for i in range(n)]
    rows = [np.concatenate([r[r == i], r[r != i]])[:length] for i, r in enumerate(rows)]
    # (the first entries of complete rows: not symmetric)
    rp = np.concatenate([[0], np.cumsum([len(r) for r in rows])]).astype(np.int32)

    def status(cols, **opts):
        try:
            rcm.order(torch.from_numpy(rp).cuda(),
                      torch.from_numpy(np.concatenate(cols).astype(np.int32)).cuda(),
                      mode=2, **opts)
        except rcm.RcmError as e:
            return e.status
        return rcm.OK

    rng = np.random.default_rng(length)
    for at in range(length - 1):
        bad = [r.copy() for r in rows]
        row = int(rng.integers(n))
        order = rng.permutation(len(bad[row]))
        bad[row] = bad[row][order]
        other = int(rng.integers(len(bad[row]) - 1))
        other += other >= at
        bad[row][at] = bad[row][other]
        assert status(bad) == rcm.ERR_BAD_CSR, (row, at, other)
    out = [r.copy() for r in rows]
    out[-1][-1] = n
    assert status(out) == rcm.ERR_BAD_CSR
    if length < n:
        assert status(rows, check_full=True) == rcm.ERR_NOT_SYMMETRIC


@pytest.mark.parametrize("case", range(6))
def test_more_vertices_than_the_records_fit(case):
    """Short rows, up to the most vertices the engine takes; runs of isolated
    vertices before, between and after the others."""
    rng = np.random.default_rng(case)
    if case == 0:
        g = I.grid2d(79, 81, seed=1)
    elif case == 1:
        g = I.strip_drop(5, 1300, 0.02, seed=2)
    elif case == 2:
        g = I.random_tree(7900, 3)
    elif case == 3:
        # (a few long rows among 8,191 vertices, most of them isolated)
        u, v = rng.integers(3000, 5000, 6000), rng.integers(3000, 5000, 6000)
        g = I.from_edges(8191, u[u != v], v[u != v], diag=False, name="isolated_8191")
    elif case == 4:
        g = I.from_edges(8191, np.zeros(0, np.int64), np.zeros(0, np.int64), name="none_8191")
    else:
        u = rng.integers(0, 8190, 3000)
        g = I.from_edges(8191, u, u + 1, diag=False, name="pairs_8191")
    _check(g)
    _check(g, reverse_mode=1, pp_variant=1)


@pytest.mark.parametrize("named", [1, 7, 64, 65, 700])
@pytest.mark.parametrize("apart", [0, 1, 6, 900])
def test_vertices_that_only_other_rows_name(named, apart):
    """Leaves of a path's middle whose own rows are empty, between isolated
    vertices: they belong to the path's component and are ordered once.  (No
    traversal of whole components meets an error in that.)"""
    n = 2000
    i = np.arange(n - 1)
    hub = np.arange(12)  # a long row
    total = n + 12 + 2 * apart + named
    leaves = n + 12 + apart + np.arange(named)
    u = np.concatenate([i, np.full(12, 20), n // 3 + np.arange(named)])
    v = np.concatenate([i + 1, n + hub, leaves])
    g = I.from_edges(total, u, v)
    rows = np.repeat(np.arange(total), np.diff(g.rowptr))
    keep = (rows < leaves[0]) | (rows > leaves[-1]) | (rows == g.colidx)
    g = I.Graph(total, np.concatenate([[0], np.cumsum(np.bincount(rows[keep], minlength=total))])
                .astype(np.int32), g.colidx[keep], f"named_{named}_{apart}")
    _check(g)
    _check(g, pp_variant=1, reverse_mode=1)

"""What a level of the component engine says beside its number of vertices: a
row longer than the row copy's eight entries, found many at a time on the
first level that holds any; more children than a level may have, met by many
rows.  Neither must depend on how many there are, nor be taken for a number of
vertices or for each other.  Whole numbers throughout: every result must equal
the oracle's."""

import numpy as np
import pytest

import oracle
from paper_1610_08128_amd import inputs as I

pytestmark = pytest.mark.gpu

COUNTS = [127, 128, 129, 255, 256, 257, 511, 512, 768, 1023, 1024]


def _fan(k, handle, *, rest=0, seed=None):
    """A path of `handle` vertices into a binary tree whose last level has k,
    each joined to nine of k more: from the path's start, k long rows come
    together.  rest: isolated vertices beside it.  Labels 0, 1, ... from the
    path's start unless a seed relabels them."""
    u, v = [np.arange(handle - 1)], [np.arange(1, handle)]
    level, n = np.array([handle - 1]), handle
    while len(level) < k:
        size = min(2 * len(level), k)
        kids = np.arange(n, n + size)
        u.append(level[np.arange(size) % len(level)])
        v.append(kids)
        level, n = kids, n + size
    for d in range(9):
        u.append(level)
        v.append(n + (np.arange(k) + d) % k)
    n += k + rest
    perm = None if seed is None else np.random.default_rng(seed).permutation(n)
    g = I.from_edges(n, np.concatenate(u), np.concatenate(v), perm=perm, name=f"fan_{k}_{handle}")
    if seed is None:
        long = np.flatnonzero(np.diff(g.rowptr) > 8)
        assert len(long) == 2 * k and np.array_equal(np.sort(level), long[:k])
    return g


def _check(g, **opts):
    import torch
    from paper_1610_08128_amd import rcm

    print(f"case {g.name} n={g.n} nnz={g.nnz} {opts}", flush=True)
    want = oracle.rcm(g.n, g.rowptr, g.colidx, **opts)
    assert want.status == oracle.OK
    perm, iperm, st = rcm.order(torch.from_numpy(g.rowptr).cuda(),
                                torch.from_numpy(g.colidx).cuda(), return_iperm=True, **opts)
    assert np.array_equal(perm.cpu().numpy(), want.perm)
    assert np.array_equal(iperm.cpu().numpy(), want.iperm)
    assert st == want.stats


def _check_batch(graphs, **opts):
    import torch
    from paper_1610_08128_amd import rcm

    vo, no, rp, ci = I.concat_batch(graphs)
    print(f"batch {[g.name for g in graphs]} {opts}", flush=True)
    perm, stats = rcm.order_batched(vo, no, torch.from_numpy(rp).cuda(),
                                    torch.from_numpy(ci).cuda(), **opts)
    perm = perm.cpu().numpy()
    for i, g in enumerate(graphs):
        want = oracle.rcm(g.n, g.rowptr, g.colidx, **opts)
        assert np.array_equal(perm[vo[i]:vo[i + 1]], want.perm), (i, g.name)
        assert stats[i] == want.stats, (i, g.name)


@pytest.mark.parametrize("k", COUNTS)
def test_component_engine(k):
    """Vertex 0's component (of so many levels that it is renumbered, and of
    few), one beside it, and components of a batch.  More than 8,191 vertices
    in a single graph, past the engines for small ones."""
    g = _fan(k, 8200)
    _check(g)
    _check(_fan(k, 300, rest=8000))
    _check(_fan(k, 300, rest=8000, seed=k), pp_variant=1, reverse_mode=1)
    _check(I.disjoint_union([I.path(5), g, _fan(k, 60)]))
    _check_batch([_fan(k, 40), I.grid2d(9, 7, seed=2), g, _fan(k, 300, seed=k)])


@pytest.mark.parametrize("k", [127, 128, 129, 200, 255, 256, 257])
def test_long_probe(k):
    """The same in a graph past the component engine's range, whose first
    structure one work-group measures (levels of at most 256 vertices)."""
    g = _fan(k, 300, rest=1 << 19)
    _check(g)
    _check(g, pp_variant=1, reverse_mode=1)


def _wide_from_one_side(children, tail, seed=None):
    """1,000 parents joined to the same children: through the vertex that
    half the children hang on, no level is wider than the parents or half the
    children; through the one the parents hang on, all children are a level.
    Label 0 behind the first, a longer path away from it than the other's."""
    parents = 1000
    half = children // 2
    x, y = tail, 5  # path 0 .. x - 1 (0 next to the first vertex), path of y
    side, top = x, x + 1
    a = np.arange(parents) + x + 2
    b = np.arange(children) + x + 2 + parents
    far = np.arange(y) + x + 2 + parents + children
    u = [np.arange(x - 1), [0], np.full(half, side), np.repeat(a, children), a, [top], far[:-1]]
    v = [np.arange(1, x), [side], b[:half], np.tile(b, parents), np.full(parents, top), [far[0]],
         far[1:]]
    n = int(far[-1]) + 1
    perm = None
    if seed is not None:  # label 0 stays
        perm = np.concatenate([[0], 1 + np.random.default_rng(seed).permutation(n - 1)])
    return I.from_edges(n, np.concatenate([np.asarray(e, dtype=np.int64) for e in u]),
                        np.concatenate([np.asarray(e, dtype=np.int64) for e in v]), perm=perm,
                        name=f"wide_{children}")


@pytest.mark.parametrize("children", [2000, 2048, 2049, 2100])
def test_only_the_labelled_level_is_wide(children):
    """The searches see half the children at once, the labelled BFS all of
    them, in rows of so many entries that 16,000 wave calls meet the level
    that is given up: the component must go to the team kernel.  Vertex 0's
    component, one beside it, and one of a batch."""
    g = _wide_from_one_side(children, 9000)
    _check(g)
    _check(_wide_from_one_side(children, 9000, seed=children))
    _check(I.disjoint_union([I.path(5), g]), reverse_mode=1)
    _check_batch([I.path(9), _wide_from_one_side(children, 100), I.grid2d(9, 7, seed=2)])


@pytest.mark.parametrize("leaves", [520, 2047, 2048, 2049, 2500])
def test_search_levels_of_long_rows(leaves):
    """Two hundred hubs joined to the same leaves: more rows than the
    work-group's list of long ones takes, on a level that is known to be too
    wide, or not, before the last of them is read."""
    hubs, tail = 200, 9000
    a = np.arange(hubs) + 1
    b = np.arange(leaves) + 1 + hubs
    far = np.arange(tail) + 1 + hubs + leaves
    u = np.concatenate([np.zeros(hubs, np.int64), np.repeat(a, leaves), [0], far[:-1]])
    v = np.concatenate([a, np.tile(b, hubs), far])
    n = int(far[-1]) + 1
    g = I.from_edges(n, u, v, perm=np.random.default_rng(leaves).permutation(n),
                     name=f"hubs_{leaves}")
    _check(g)
    _check_batch([I.path(9), g], pp_variant=1)

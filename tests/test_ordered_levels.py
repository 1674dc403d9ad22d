"""The team kernel's labelled levels with one barrier (claims by ordered keys)
where they begin, are shared out again and end: lists at and past the length
at which they go back to claims by label, levels at the narrow limit, vertices
with more children than are kept in registers, teams of every size.  Whole
numbers throughout: every result must equal the oracle's."""

import numpy as np
import pytest

import oracle
from paper_1610_08128_amd import inputs as I

pytestmark = pytest.mark.gpu


def _check(g, **opts):
    import torch
    from paper_1610_08128_amd import rcm

    print(f"case {g.name} n={g.n} nnz={g.nnz} {opts}", flush=True)
    want = oracle.rcm(g.n, g.rowptr, g.colidx, pp_variant=opts.get("pp_variant", 0),
                      reverse_mode=opts.get("reverse_mode", 0))
    assert want.status == oracle.OK
    rp = torch.from_numpy(g.rowptr).cuda()
    ci = torch.from_numpy(g.colidx).cuda()
    perm, iperm, st = rcm.order(rp, ci, return_iperm=True, mode=1, **opts)
    assert np.array_equal(perm.cpu().numpy(), want.perm), (g.name, opts)
    assert np.array_equal(iperm.cpu().numpy(), want.iperm), (g.name, opts)
    assert st == want.stats


def _regular(n, degree, seed):
    """Rows of up to `degree` off-diagonal entries, most of them children."""
    rng = np.random.default_rng(seed)
    i = np.arange(n)
    u, v = [], []
    for _ in range(degree // 2):
        p = rng.permutation(n)
        u.append(i)
        v.append(p)
    u, v = np.concatenate(u), np.concatenate(v)
    keep = u != v
    return I.from_edges(n, u[keep], v[keep], name=f"regular_{n}_{degree}_{seed}")


def _graphs():
    return [I.grid3d(24, 25, 26, seed=1), I.grid3d(40, 41, 9, seed=2), I.grid2d(180, 170, seed=3),
            I.shuffle_rows(I.drop_diagonal(I.grid3d(20, 21, 22, seed=4)), 5),
            _regular(6000, 6, 6), _regular(30000, 4, 7),
            I.disjoint_union([I.grid3d(18, 19, 20), I.grid2d(70, 60), I.path(5)], seed=8)]


@pytest.mark.parametrize("team", [2, 3, 8, 64])
@pytest.mark.parametrize("rebalance", [2, 3, 8, 1000])
def test_teams_and_shares(team, rebalance):
    """Few work-groups have long lists (and leave), many have short ones;
    narrow_cutoff -1 keeps every level on the team."""
    for i, g in enumerate(_graphs()):
        _check(g, team_size=team, label_team=team, rebalance_levels=rebalance, block_threads=256,
               narrow_cutoff=(-1, 64, 300)[i % 3], small_cutoff=1)


@pytest.mark.parametrize("threads", [256, 512])
def test_variants(threads):
    for i, g in enumerate(_graphs()):
        _check(g, team_size=16, label_team=4 + 4 * (i % 3), block_threads=threads, small_cutoff=1,
               pp_variant=i % 2, reverse_mode=1, narrow_cutoff=-1)


@pytest.mark.parametrize("width", [255, 256, 257, 511, 512, 513, 514])
def test_list_lengths(width):
    """A strip whose levels are that wide on a team of two: lists at the
    length that ends the one-barrier levels, with a hair on either side."""
    m = 60
    i = np.arange(width * m).reshape(m, width)
    u = [i[:-1].ravel(), i[0, :-1], i[0]]
    v = [i[1:].ravel(), i[0, 1:], np.roll(i[0], 7)]
    g = I.from_edges(i.size + 1, np.concatenate(u), np.concatenate(v),
                     perm=np.random.default_rng(width).permutation(i.size + 1),
                     name=f"comb_{width}")
    for team in (2, 4):
        _check(g, team_size=team, label_team=team, narrow_cutoff=-1, block_threads=256,
               small_cutoff=1)


@pytest.mark.parametrize("team", [128, 256])
@pytest.mark.parametrize("rebalance", [2, 8])
def test_keys_run_out(team, rebalance):
    """2^31 / (2,048 team) levels use up the keys: a strip of about 9,000
    levels goes back to claims by label for that reason, in the middle of its
    labelled BFS, and stays there."""
    g = I.strip_drop(8, 9000, 0.01, seed=team)
    levels = oracle.rcm(g.n, g.rowptr, g.colidx).stats["num_levels"]
    # (but for the first few, every level takes keys until they run out)
    assert levels > (1 << 31) // (team << 11) + 500
    _check(g, team_size=team, label_team=team, rebalance_levels=rebalance, block_threads=256,
           narrow_cutoff=-1, small_cutoff=1, relabel_levels=-1)


def _one_way(seed, side, tail, at):
    """A 3D grid between two paths, and from the second path to the grid's
    middle an arc without its way back, which every search but one from the
    second path's end passes too late."""
    m = side ** 3
    c = np.arange(m).reshape(side, side, side)
    a, b = np.arange(tail) + m, np.arange(tail) + m + tail
    u = [c[:-1].ravel(), c[:, :-1].ravel(), c[:, :, :-1].ravel(), [0], a[:-1], [m - 1], b[:-1]]
    v = [c[1:].ravel(), c[:, 1:].ravel(), c[:, :, 1:].ravel(), a[:1], a[1:], b[:1], b[1:]]
    n = m + 2 * tail
    perm = np.random.default_rng(seed).permutation(n)
    g = I.from_edges(n, np.concatenate(u), np.concatenate(v), perm=perm)
    row, col = perm[b[at]], perm[c[side // 2, side // 2, side // 2]]
    end = g.rowptr[row + 1]
    rowptr = g.rowptr.copy()
    rowptr[row + 1:] += 1
    return I.Graph(n, rowptr, np.insert(g.colidx, end, col).astype(np.int32),
                   f"one_way_{seed}_{side}_{at}")


@pytest.mark.parametrize("seed", range(2, 8))
@pytest.mark.parametrize("narrow", [-1, 64])
def test_arcs_back_to_ordered_levels(seed, narrow):
    """Levels labelled by keys stay as they are when later ones, by labels or
    by keys, have an arc back to them (it is no error that a traversal of
    whole components meets)."""
    for side, at in ((18, 30), (18, 2), (26, 30)):
        g = _one_way(seed, side, 300, at)
        for team, rebalance in ((4, 8), (8, 2), (64, 8)):
            _check(g, team_size=team, label_team=team, block_threads=256, narrow_cutoff=narrow,
                   rebalance_levels=rebalance, small_cutoff=1, relabel_levels=-1)

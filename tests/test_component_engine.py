"""The component engine (one work-group per component, levels in LDS) at the
sizes where it can go wrong: the level widths at which a lane's share, a scan
or a frontier changes or ends, rows at the lengths that change how they are
read, graphs at its vertex limit, and what it declines to the team kernel.
Whole numbers throughout: every result must equal the oracle's."""

import sys
import threading
import time

import numpy as np
import pytest

import oracle
from paper_1610_08128_amd import inputs as I

pytestmark = pytest.mark.gpu


def _say(msg):
    print(msg, flush=True)
    sys.stdout.flush()


def _order(g, **opts):
    import torch
    from paper_1610_08128_amd import rcm

    rp = torch.from_numpy(g.rowptr).cuda()
    ci = torch.from_numpy(g.colidx if g.colidx.size else np.zeros(1, np.int32)).cuda()
    perm, iperm, st = rcm.order(rp, ci, return_iperm=True, **opts)
    return perm.cpu().numpy(), iperm.cpu().numpy(), st


def _check(g, **opts):
    _say(f"case {g.name} n={g.n} nnz={g.nnz} {opts}")
    want = oracle.rcm(g.n, g.rowptr, g.colidx, pp_variant=opts.get("pp_variant", 0),
                      reverse_mode=opts.get("reverse_mode", 0))
    assert want.status == oracle.OK
    perm, iperm, st = _order(g, **opts)
    assert np.array_equal(perm, want.perm) and np.array_equal(iperm, want.iperm)
    assert st == want.stats


def _check_batch(graphs, **opts):
    import torch
    from paper_1610_08128_amd import rcm

    vo, no, rp, ci = I.concat_batch(graphs)
    _say(f"batch of {len(graphs)} graphs {[g.name for g in graphs][:6]} {opts}")
    perm, stats = rcm.order_batched(vo, no, torch.from_numpy(rp).cuda(),
                                    torch.from_numpy(ci).cuda(), **opts)
    perm = perm.cpu().numpy()
    for i, g in enumerate(graphs):
        want = oracle.rcm(g.n, g.rowptr, g.colidx, pp_variant=opts.get("pp_variant", 0),
                          reverse_mode=opts.get("reverse_mode", 0))
        assert np.array_equal(perm[vo[i]:vo[i + 1]], want.perm), (i, g.name)
        assert stats[i] == want.stats, (i, g.name)


def _broom(width, *, handle=7000, seed=None, extra=0):
    """A path of `handle` vertices whose end is the root of a binary tree with
    `width` vertices on its last level: the pseudo-peripheral root is the
    path's other end, so the labelled BFS meets exactly that width too.
    extra: leaves on one path vertex (a row that long)."""
    u, v = [np.arange(handle - 1)], [np.arange(1, handle)]
    level = [handle - 1]
    n = handle
    while len(level) < width:
        size = min(2 * len(level), width)
        kids = np.arange(n, n + size)
        u.append(np.asarray(level)[np.arange(size) % len(level)])
        v.append(kids)
        level = list(kids)
        n += size
    if extra:
        u.append(np.full(extra, 3))
        v.append(np.arange(n, n + extra))
        n += extra
    perm = np.random.default_rng(seed).permutation(n) if seed is not None else None
    return I.from_edges(n, np.concatenate(u), np.concatenate(v), perm=perm,
                        name=f"broom_{width}_x{extra}")


WIDTHS = [1, 63, 64, 65, 127, 128, 129, 255, 256, 257, 511, 512, 513, 1023, 1024, 1025]


@pytest.mark.parametrize("width", WIDTHS)
@pytest.mark.parametrize("copy", ["1", "0"])
def test_level_widths(width, copy, monkeypatch):
    """On the row copy and on the CSR (RCM_ELL=0); past 1,024 the team kernel
    takes over."""
    monkeypatch.setenv("RCM_ELL", copy)
    _check(_broom(width, seed=width))
    _check(_broom(width), pp_variant=1, reverse_mode=1)


@pytest.mark.parametrize("width", [1023, 1024, 1025, 1536, 2047, 2048, 2049])
def test_level_widths_batched(width):
    """A batch goes on to the CSR for levels too wide for the rows' copy, and
    to the team kernel past 2,048."""
    graphs = [_broom(width, handle=300, seed=width), I.path(5),
              _broom(width, handle=50), I.rgg_patches(2000, width), I.path(1)]
    _check_batch(graphs)
    _check_batch(graphs, pp_variant=1, reverse_mode=1)


@pytest.mark.parametrize("row", [7, 8, 9, 16, 17, 33, 511, 512, 513, 1500])
def test_row_lengths(row):
    """A long row in a graph of short ones, alone and in a batch (whose
    components decide for themselves between the rows' copy and the CSR)."""
    g = _broom(40, seed=row, extra=row)
    _check(g)
    _check(I.shuffle_rows(I.drop_diagonal(g), row), reverse_mode=1)
    _check_batch([_broom(12, handle=60, seed=1), _broom(9, handle=80, seed=row, extra=row),
                  I.grid2d(9, 7, seed=2)])


def test_many_long_rows_in_one_level():
    """More rows longer than 512 entries in one level than its list holds:
    the others are read by their lanes."""
    hubs, leaves = 40, 560
    u = [np.zeros(hubs, np.int64)]
    v = [np.arange(1, hubs + 1)]
    for h in range(hubs):  # every hub joined to the same leaves
        u.append(np.full(leaves, 1 + h))
        v.append(np.arange(hubs + 1, hubs + 1 + leaves))
    n = hubs + 1 + leaves
    tail = np.arange(n, n + 7000)
    u += [np.array([0]), tail[:-1]]
    v += [tail[:1], tail[1:]]
    g = I.from_edges(n + 7000, np.concatenate(u), np.concatenate(v), name="hubs_40x560",
                     perm=np.random.default_rng(4).permutation(n + 7000))
    _check(g)
    _check(g, pp_variant=1)
    _check_batch([g, I.path(9)])


@pytest.mark.parametrize("extra", [0, 1])
def test_vertex_limit(extra):
    """2^19 vertices (its visited bitmap's size) and one more."""
    g = I.grid2d(256, 2048, seed=3)
    assert g.n == 1 << 19
    if extra:
        g = I.disjoint_union([g, I.path(1)])
        g.name = "grid2d_256x2048_plus1"
    _check(g, relabel_levels=-1)


def test_components_beside_the_probed_one():
    """Vertex 0's component resumed together with the others: it alone, the
    largest, the smallest, an isolated vertex; wide ones among them."""
    a, b = I.grid2d(80, 90, seed=1), I.rgg_patches(9000, 2)
    wide = I.grid3d(38, 38, 38, seed=3)
    for parts in ([a, b], [I.path(1), a, b], [I.path(3), wide, I.path(1), a], [wide, b],
                  [b, wide, I.relabel(I.star(9000), 5)[0]]):
        g = I.disjoint_union(parts)
        g.name = "union_" + "_".join(p.name for p in parts)
        _check(g)
        _check(g, pp_variant=1, reverse_mode=1)
        _check(I.disjoint_union(parts, seed=7))


def test_long_components_with_and_without_renumbering():
    """A component of 4,096 levels or more is renumbered after the probe and
    finished by the window engine; rows too long for that stay."""
    from paper_1610_08128_amd import rcm

    _check(I.strip_drop(8, 6000, 0.01, seed=5))
    assert rcm.last_timings()["used_mode"] == 4
    _check(I.disjoint_union([I.strip_drop(8, 6000, 0.01, seed=5), I.grid2d(40, 40, seed=6)]),
           pp_variant=1)
    assert rcm.last_timings()["used_mode"] == 4
    for g in (I.strip_drop(8, 6000, 0.01, seed=5), I.path(20000, seed=8)):
        _check(g, relabel_levels=-1)
        assert rcm.last_timings()["used_mode"] == 1
    _check(I.grid3d(4, 4, 5000, seed=9))  # rows of up to 6: the window engine declines
    assert rcm.last_timings()["used_mode"] == 1


def test_asymmetric_patterns_are_reported():
    from paper_1610_08128_amd import rcm

    def drop(g, r, c):
        a, b = g.rowptr[r], g.rowptr[r + 1]
        k = a + int(np.nonzero(g.colidx[a:b] == c)[0][0])
        rp = g.rowptr.copy()
        rp[r + 1:] -= 1
        return I.Graph(g.n, rp, np.delete(g.colidx, k), g.name + "_asym")

    path = I.path(8000)  # its end loses the way back
    for g in (drop(path, 7999, 7998), drop(I.disjoint_union([I.path(9), path]), 8008, 8007)):
        _say(f"case {g.name} n={g.n}")
        with pytest.raises(rcm.RcmError) as e:
            _order(g, relabel_levels=-1)
        assert e.value.status == rcm.ERR_NOT_SYMMETRIC


def test_shuffled_tasks_and_abort_in_flight():
    from paper_1610_08128_amd import rcm

    graphs = [I.grid2d(40 + i, 30, seed=i) for i in range(6)] + [I.rgg_patches(3000, 4),
                                                                 I.path(1), I.star(7)]
    for seed in (1, 0xBEEF):
        _check_batch(graphs, shuffle_seed=seed)
    g = I.path(400_000, seed=1)
    with rcm.AbortFlag() as flag:
        t0 = time.perf_counter()
        want = _order(g, abort_flag=flag, relabel_levels=-1)
        full = time.perf_counter() - t0
        assert full > 0.2, "too short to abort in flight"
        timer = threading.Timer(full / 4, flag.set)
        timer.start()
        try:
            t0 = time.perf_counter()
            with pytest.raises(rcm.RcmError) as e:
                _order(g, abort_flag=flag, relabel_levels=-1)
            took = time.perf_counter() - t0
        finally:
            timer.join()
        assert e.value.status == rcm.ERR_ABORTED
        assert took < full * 5 / 8
        flag.clear()
        again = _order(g, abort_flag=flag, relabel_levels=-1)
    assert all(np.array_equal(x, y) for x, y in zip(want[:2], again[:2])) and want[2] == again[2]


@pytest.mark.parametrize("n", [1, 2, 127, 128, 129, 1023, 1025, 16384, 16385])
@pytest.mark.parametrize("copy", ["1", "0"])
def test_statistics_of_the_result(n, copy, monkeypatch):
    """Bandwidth and profile of the result, read from the row copy or the
    CSR, at the edges of their tiles of 128 rows and 16,384 sums, with rows of
    the diagonal alone, of one and of many entries."""
    monkeypatch.setenv("RCM_ELL", copy)
    rng = np.random.default_rng(n)
    u = rng.integers(0, n, n // 2)
    v = rng.integers(0, n, n // 2)
    keep = u != v
    g = I.from_edges(n, u[keep], v[keep], name=f"sparse_{n}")
    _check(g, mode=1)
    if n > 2:
        _check(I.from_edges(n, np.zeros(n - 1, np.int64), np.arange(1, n), diag=False,
                            perm=rng.permutation(n), name=f"star_{n}"), mode=1)

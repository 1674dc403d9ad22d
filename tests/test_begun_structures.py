"""First level structures that the component engine's probe (or, past its
range, the long probe) begins and declines, which the team kernel goes on
with: long narrow parts into wide ones or into long rows, vertex 0 at either
end and between, at the number of levels from which the way is kept.  Whole
numbers throughout: every result must equal the oracle's."""

import numpy as np
import pytest

import oracle
from paper_1610_08128_amd import inputs as I

pytestmark = pytest.mark.gpu


def _handle(length, g, start, seed, rest=0):
    """A path of `length` vertices hung on g's vertex 0; label 0 at the path's
    end, its middle or in g's last vertex; isolated vertices beside."""
    r = np.repeat(np.arange(g.n), np.diff(g.rowptr))
    keep = r < g.colidx
    p = np.arange(length) + g.n
    u = np.concatenate([r[keep], p[:-1], [0]])
    v = np.concatenate([g.colidx[keep], p[1:], p[:1]])
    n = g.n + length + rest
    perm = np.random.default_rng(seed).permutation(n)
    at = {"end": p[-1], "middle": p[length // 2], "far": g.n - 1}[start]
    other = int(np.flatnonzero(perm == 0)[0])
    perm[at], perm[other] = perm[other], perm[at]
    return I.from_edges(n, u, v, perm=perm, name=f"handle_{length}_{g.name}_{start}")


def _check(g, **opts):
    import torch
    from paper_1610_08128_amd import rcm

    print(f"case {g.name} n={g.n} nnz={g.nnz} {opts}", flush=True)
    want = oracle.rcm(g.n, g.rowptr, g.colidx, **{k: v for k, v in opts.items() if k in
                                                  ("pp_variant", "reverse_mode")})
    assert want.status == oracle.OK
    perm, iperm, st = rcm.order(torch.from_numpy(g.rowptr).cuda(),
                                torch.from_numpy(g.colidx).cuda(), return_iperm=True, **opts)
    assert np.array_equal(perm.cpu().numpy(), want.perm)
    assert np.array_equal(iperm.cpu().numpy(), want.iperm)
    assert st == want.stats


def _sparse(n, seed):
    """A random graph of mean degree 4: rows past eight entries, wide levels."""
    rng = np.random.default_rng(seed)
    u, v = rng.integers(0, n, 2 * n), rng.integers(0, n, 2 * n)
    keep = u != v
    t = I.random_tree(n, seed)  # connected
    r = np.repeat(np.arange(n), np.diff(t.rowptr))
    return I.from_edges(n, np.concatenate([u[keep], r]), np.concatenate([v[keep], t.colidx]),
                        name=f"sparse_{n}")


PARTS = [lambda: I.grid3d(40, 41, 42), lambda: _sparse(30000, 1), lambda: I.star(5000),
         lambda: I.disjoint_union([I.grid3d(40, 41, 42), I.grid2d(70, 80)])]


@pytest.mark.parametrize("part", range(len(PARTS)))
@pytest.mark.parametrize("length", [1, 20, 31, 32, 33, 34, 400, 5000])
def test_component_range(part, length):
    g = PARTS[part]()
    for start in ("end", "middle", "far"):
        h = _handle(length, g, start, length, rest=7000 if g.n < 9000 else 3)
        _check(h)
        if length in (33, 5000):
            _check(h, pp_variant=1, reverse_mode=1)
            _check(h, relabel_levels=-1)


@pytest.mark.parametrize("part", range(2))
@pytest.mark.parametrize("length", [31, 33, 300, 5000])
def test_past_the_component_range(part, length):
    """The long probe: levels of at most 256 vertices, bounded rows."""
    g = (I.grid3d(40, 41, 42), _sparse(30000, 1))[part]
    for start in ("end", "middle", "far"):
        h = _handle(length, g, start, length, rest=(1 << 19) + 5)
        _check(h)
        if length == 5000:
            _check(h, pp_variant=1, reverse_mode=1)


def test_shuffled_teams():
    for seed in (1, 77):
        _check(_handle(900, I.grid3d(40, 41, 42), "end", seed), shuffle_seed=seed)

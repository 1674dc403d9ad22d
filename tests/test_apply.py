"""Applying an ordering: the oracle's B = P A P^T and y = A x are pinned to
library routines and to the ordering's own statistics (CPU); the GPU's
permuted matrix equals the oracle's exactly and its product agrees within
the float64 rounding bound (GPU)."""

import numpy as np
import pytest
import scipy.linalg
import scipy.sparse as sp

import oracle
from paper_1610_08128_amd import inputs as I


def _graphs():
    return [I.grid2d(9, 13, seed=3), I.rgg_patches(300, 5), I.path(7, seed=2),
            I.add_random_self_loops(I.random_tree(60, 4), 0.3, 4),
            I.disjoint_union([I.complete(5), I.grid3d(3, 4, 2, seed=1)], seed=9),
            # rows around and well past the register-sort limit of the
            # permutation (16 entries), and a very long star row
            I.disjoint_union([I.complete(16), I.complete(17), I.star(40), I.path(3)], seed=5),
            I.erdos_renyi(120, 0.2, 6)]


def _csr(g, vals=None):
    data = np.ones(g.nnz) if vals is None else vals
    return sp.csr_matrix((data, g.colidx, g.rowptr), shape=(g.n, g.n))


@pytest.mark.parametrize("gi", range(7))
def test_oracle_permute_matches_scipy_indexing(gi):
    g = _graphs()[gi]
    rng = np.random.default_rng(gi)
    vals = rng.standard_normal(g.nnz)
    perm = oracle.rcm(g.n, g.rowptr, g.colidx).perm
    rp, ci, v = oracle.permute_csr(g.n, g.rowptr, g.colidx, perm, vals)
    want = _csr(g, vals)[perm][:, perm].tocsr()
    want.sort_indices()
    assert np.array_equal(rp, want.indptr) and np.array_equal(ci, want.indices)
    assert np.array_equal(v, want.data)


@pytest.mark.parametrize("gi", range(7))
def test_oracle_permute_gives_the_reported_bandwidth(gi):
    # the bandwidth of the permuted pattern (library routine on the dense
    # matrix with the diagonal present) is the ordering's bandwidth_after
    g = _graphs()[gi]
    r = oracle.rcm(g.n, g.rowptr, g.colidx)
    rp, ci, _ = oracle.permute_csr(g.n, g.rowptr, g.colidx, r.perm)
    dense = sp.csr_matrix((np.ones(ci.size), ci, rp), shape=(g.n, g.n)).toarray()
    dense[np.arange(g.n), np.arange(g.n)] = 1.0
    lo, hi = scipy.linalg.bandwidth(dense)
    assert max(lo, hi) == r.stats["bandwidth_after"]


def test_oracle_permute_identity_and_round_trip():
    g = I.rgg_patches(200, 3)
    ident = np.arange(g.n, dtype=np.int32)
    rp, ci, _ = oracle.permute_csr(g.n, g.rowptr, g.colidx, ident)
    want = _csr(g)
    want.sort_indices()
    assert np.array_equal(rp, want.indptr) and np.array_equal(ci, want.indices)
    perm = np.random.default_rng(1).permutation(g.n).astype(np.int32)
    inv = np.empty_like(perm)
    inv[perm] = np.arange(g.n, dtype=np.int32)
    rp1, ci1, _ = oracle.permute_csr(g.n, g.rowptr, g.colidx, perm)
    rp2, ci2, _ = oracle.permute_csr(g.n, rp1, ci1, inv)
    assert np.array_equal(rp2, want.indptr) and np.array_equal(ci2, want.indices)


def test_oracle_spmv_matches_scipy():
    g = I.grid3d(5, 6, 7, seed=2)
    rng = np.random.default_rng(0)
    vals = rng.standard_normal(g.nnz)
    x = rng.standard_normal(g.n)
    y = oracle.spmv(g.n, g.rowptr, g.colidx, x, vals)
    assert np.allclose(y, _csr(g, vals) @ x, rtol=1e-14, atol=1e-14)
    y1 = oracle.spmv(g.n, g.rowptr, g.colidx, x)
    assert np.allclose(y1, _csr(g) @ x, rtol=1e-14, atol=1e-14)


@pytest.mark.gpu
@pytest.mark.parametrize("gi", range(7))
def test_gpu_permute_and_spmv(gi):
    import torch
    from paper_1610_08128_amd import apply, rcm

    g = _graphs()[gi]
    rng = np.random.default_rng(10 + gi)
    vals = rng.standard_normal(g.nnz)
    x = rng.standard_normal(g.n)
    rp = torch.from_numpy(g.rowptr).cuda()
    ci = torch.from_numpy(g.colidx).cuda()
    perm, iperm, st = rcm.order(rp, ci, return_iperm=True)
    want_rp, want_ci, want_v = oracle.permute_csr(g.n, g.rowptr, g.colidx, perm.cpu().numpy(), vals)
    vd = torch.from_numpy(vals).cuda()
    brp, bci, bv = apply.permute(rp, ci, perm, iperm, vd)
    assert np.array_equal(brp.cpu().numpy(), want_rp)
    assert np.array_equal(bci.cpu().numpy(), want_ci)
    assert np.array_equal(bv.cpu().numpy(), want_v)  # values are moved, not computed
    brp2, bci2, _ = apply.permute(rp, ci, perm, iperm)
    assert np.array_equal(bci2.cpu().numpy(), want_ci)
    # product: each |y_i - y'_i| <= 2 * L_i * u * sum_j |a_ij x_j| for row length L_i
    # (two summation orders, each within L_i * u of the exact sum); u = 2^-53
    y = apply.spmv(brp, bci, torch.from_numpy(x).cuda(), bv).cpu().numpy()
    want_y = oracle.spmv(g.n, want_rp, want_ci, x, want_v)
    L = np.diff(want_rp).astype(np.float64)
    absum = oracle.spmv(g.n, want_rp, want_ci, np.abs(x), np.abs(want_v))
    assert np.all(np.abs(y - want_y) <= 2 * L * 2.0**-53 * absum + 1e-300)
    # the permuted pattern's bandwidth is the one the ordering reported
    rows = np.repeat(np.arange(g.n), np.diff(want_rp))
    bw = int(np.max(np.maximum(rows - want_ci, 0))) if want_ci.size else 0
    assert bw == st["bandwidth_after"]


def _check_gpu_permute(g, seed):
    import torch
    from paper_1610_08128_amd import apply, rcm

    rng = np.random.default_rng(seed)
    vals = rng.standard_normal(g.nnz)
    rp = torch.from_numpy(g.rowptr).cuda()
    ci = torch.from_numpy(g.colidx).cuda()
    perm, iperm, _ = rcm.order(rp, ci, return_iperm=True)
    want_rp, want_ci, want_v = oracle.permute_csr(g.n, g.rowptr, g.colidx, perm.cpu().numpy(),
                                                  vals)
    brp, bci, bv = apply.permute(rp, ci, perm, iperm, torch.from_numpy(vals).cuda())
    assert np.array_equal(brp.cpu().numpy(), want_rp)
    assert np.array_equal(bci.cpu().numpy(), want_ci)
    assert np.array_equal(bv.cpu().numpy(), want_v)


@pytest.mark.gpu
def test_gpu_permute_dense_rows():
    """About 60 entries per row: a block's 256 rows then hold more entries than
    its LDS stage, so the rows are written directly; rows in random order."""
    g = I.shuffle_rows(I.erdos_renyi(600, 0.1, 11), 2)
    assert int(g.rowptr[256]) > 256 * 16
    _check_gpu_permute(g, 1)


@pytest.mark.gpu
def test_gpu_permute_many_tiles():
    """More rows than one pass of the grid covers (8,192 blocks of 256 rows),
    so blocks take a second tile."""
    g = I.grid2d(1500, 1500, seed=12)
    assert g.n > 8192 * 256
    _check_gpu_permute(g, 2)


@pytest.mark.gpu
def test_gpu_permute_long_rows():
    """Rows longer than a register sort: rows of 17 to 300 entries, and hub
    rows of exactly the LDS sort's 8,192 entries, one more, and 20,001 (the
    last two sort in the scratch array), with rows in random order."""
    g = I.shuffle_rows(I.disjoint_union([I.star(20001), I.star(8192), I.star(8193),
                                         I.erdos_renyi(900, 0.15, 13), I.star(18), I.star(300)],
                                        seed=14), 3)
    lens = np.diff(g.rowptr)
    assert {8192, 8193, 20001} <= set(lens.tolist())
    _check_gpu_permute(g, 4)


def _rows_of(lengths, seed):
    """A matrix (any pattern: the calls below do not need symmetry) whose row
    i holds lengths[i] distinct columns in random order."""
    rng = np.random.default_rng(seed)
    n = len(lengths)
    rowptr = np.concatenate([[0], np.cumsum(lengths)]).astype(np.int32)
    cols = [rng.permutation(n)[:k] for k in lengths]
    colidx = np.concatenate(cols).astype(np.int32) if n else np.zeros(0, np.int32)
    return I.Graph(n, rowptr, colidx, "rows")


# every length at which a row changes hands (a lane's second entry, a wave, a
# work-group), matrices of one tile of 128 rows, one row less and more, and a
# few tiles; with and without empty rows
@pytest.mark.gpu
@pytest.mark.parametrize("n", [1, 7, 127, 128, 129, 1025, 4099])
@pytest.mark.parametrize("values", [True, False])
def test_gpu_permute_and_spmv_row_lengths(n, values):
    import torch
    from paper_1610_08128_amd import apply

    rng = np.random.default_rng(n)
    kinds = [[0, 1, 7, 8, 9, 15, 16, 17, 33, 63, 64, 65, 200], [5, 7], [0, 0, 3], [8, 9, 16],
             [12, 17, 28]]
    for i, kind in enumerate(kinds):
        lengths = np.minimum(rng.choice(kind, n), n)
        g = _rows_of(lengths, 100 * n + i)
        print(f"case n={n} kind={kind} nnz={g.nnz}", flush=True)
        perm = rng.permutation(n).astype(np.int32)
        iperm = np.empty_like(perm)
        iperm[perm] = np.arange(n, dtype=np.int32)
        vals = rng.standard_normal(g.nnz) if values else None
        want = oracle.permute_csr(g.n, g.rowptr, g.colidx, perm, vals)
        dev = [torch.from_numpy(t).cuda() if t is not None else None
               for t in (g.rowptr, g.colidx, perm, iperm, vals)]
        got = apply.permute(*dev)
        assert np.array_equal(got[0].cpu().numpy(), want[0])
        assert np.array_equal(got[1].cpu().numpy(), want[1])
        if values:
            assert np.array_equal(got[2].cpu().numpy(), want[2])
        # two summation orders of a row of L terms: each within L u of the
        # exact sum, u = 2^-53
        x = rng.standard_normal(n)
        y = apply.spmv(dev[0], dev[1], torch.from_numpy(x).cuda(), dev[4]).cpu().numpy()
        exact = oracle.spmv(g.n, g.rowptr, g.colidx, x, vals)
        total = oracle.spmv(g.n, g.rowptr, g.colidx, np.abs(x),
                            np.abs(vals) if values else None)
        assert np.all(np.abs(y - exact) <= 2 * lengths * 2.0**-53 * total)


@pytest.mark.gpu
@pytest.mark.parametrize("n", [1, 127, 129, 1000])
@pytest.mark.parametrize("values", [True, False])
def test_gpu_permute_arrays_longer_than_the_matrix(n, values):
    """Column and value arrays with room past the matrix's last entry, whose
    words there are no columns: no row may look at them, an empty one at the
    matrix's end least of all."""
    import torch
    from paper_1610_08128_amd import apply

    rng = np.random.default_rng(n)
    lengths = rng.integers(0, min(n, 20) + 1, n)
    lengths[-(n // 3 + 1):] = 0
    g = _rows_of(lengths, n)
    vals = rng.standard_normal(g.nnz)
    perm = rng.permutation(n).astype(np.int32)
    iperm = np.argsort(perm).astype(np.int32)
    want_rp, want_ci, want_v = oracle.permute_csr(n, g.rowptr, g.colidx, perm, vals)
    room = 37
    ci = np.concatenate([g.colidx, np.full(room, 1 << 30, np.int32)])
    v = np.concatenate([vals, np.full(room, np.nan)])
    brp, bci, bv = apply.permute(
        torch.from_numpy(g.rowptr).cuda(), torch.from_numpy(ci).cuda(),
        torch.from_numpy(perm).cuda(), torch.from_numpy(iperm).cuda(),
        torch.from_numpy(v).cuda() if values else None)
    assert np.array_equal(brp.cpu().numpy(), want_rp)
    assert np.array_equal(bci.cpu().numpy()[:g.nnz], want_ci)
    assert not values or np.array_equal(bv.cpu().numpy()[:g.nnz], want_v)


def _permute_workspace(n, nnz, values):
    """The interface's size: degrees, the scan's sums, a copy of the columns
    and of the values, sort pairs, each rounded up to 256 bytes."""
    up = lambda b: (b + 255) // 256 * 256  # noqa: E731
    return (up(4 * n) + up(4 * (n // 4096 + 2)) + up(4 * nnz) + (up(8 * nnz) if values else 0)
            + up(8 * nnz))


@pytest.mark.parametrize("n", [1, 64, 4095, 4096, 100_000, 2**31 - 1])
def test_permute_workspace_is_the_interfaces(n):
    from paper_1610_08128_amd import apply

    for nnz in (0, 1, 63, n // 3, n - 1, n, n + 63, n + 64, n + 65, 7 * n, 2**31 - 2):
        if nnz >= 2**31 - 1:
            continue
        for values in (False, True):
            assert apply.permute_workspace_bytes(n, nnz, values) == \
                _permute_workspace(n, nnz, values)


@pytest.mark.gpu
@pytest.mark.parametrize("entries", [0, 1, 70, 1000, 9000, 12_000, 13_000, 37_000])
@pytest.mark.parametrize("values", [True, False])
def test_gpu_permute_few_entries(entries, values):
    """Fewer entries than rows, around the numbers at which the workspace has
    no room for the rows' begins; short, medium and long rows among them, and
    nothing behind the workspace touched."""
    import torch
    from paper_1610_08128_amd import apply

    n = 12_500
    rng = np.random.default_rng(entries)
    lengths = np.zeros(n, np.int64)
    left = entries
    for k in (8200, 300, 40, 17, 9):
        if left >= k:
            lengths[rng.integers(0, n // 2)] = k
            left = entries - int(lengths.sum())
    lengths[n // 2:] += rng.multinomial(left, np.full(n - n // 2, 1 / (n - n // 2)))
    g = _rows_of(lengths, entries)
    assert g.nnz == entries
    vals = rng.standard_normal(entries)
    perm = rng.permutation(n).astype(np.int32)
    iperm = np.argsort(perm).astype(np.int32)
    want_rp, want_ci, want_v = oracle.permute_csr(n, g.rowptr, g.colidx, perm, vals)
    size = _permute_workspace(n, entries, values)
    buf = torch.full((size + 4096,), 0x5A, dtype=torch.uint8, device="cuda")
    args = [torch.from_numpy(a).cuda() for a in (g.rowptr, g.colidx, perm, iperm)]
    v = torch.from_numpy(vals).cuda() if values else None
    with pytest.raises(Exception):
        apply.permute(*args, v, workspace=buf[:size - 1])
    brp, bci, bv = apply.permute(*args, v, workspace=buf[:size])
    assert np.array_equal(brp.cpu().numpy(), want_rp)
    assert np.array_equal(bci.cpu().numpy(), want_ci)
    assert not values or np.array_equal(bv.cpu().numpy(), want_v)
    assert bool((buf[size:] == 0x5A).all())


def _blocks_of_rows(n, seed):
    """Rows in stretches of 300 of a kind, so that waves meet each alone and
    next to others: none, few and two batches of entries, rows at the lengths
    at which a wave goes on by other means, a few long ones among short."""
    rng = np.random.default_rng(seed)
    kinds = [(5,), (16,), (17,), (0,), (0, 3), (1, 30), (64,), (65,), (100,), (6, 6, 6, 150),
             (6,) * 40 + (3000,), (72, 128, 129), (8, 9), (20, 0, 500), (192, 193, 0), (63, 64)]
    lengths = np.concatenate([rng.choice(kinds[i % len(kinds)] if i < 40 else (0, 1, 2, 5, 7), 300)
                              for i in range(n // 300 + 1)])[:n]
    rowptr = np.concatenate([[0], np.cumsum(lengths)]).astype(np.int32)
    return rowptr, rng.integers(0, n, int(rowptr[-1])).astype(np.int32)


# the product's numbers of rows in flight change at 2^18 and 2^19 rows
@pytest.mark.gpu
@pytest.mark.parametrize("n", [5000, 2**18 - 1, 2**18, 2**19 - 1, 2**19, 2**19 + 333])
@pytest.mark.parametrize("values", [True, False])
def test_gpu_spmv_kinds_of_rows(n, values):
    """Each |y_i - y'_i| <= 2 * L_i * u * sum_j |a_ij x_j| (two summation orders,
    each within L_i * u of the exact sum); u = 2^-53."""
    import torch
    from paper_1610_08128_amd import apply

    rowptr, colidx = _blocks_of_rows(n, n)
    rng = np.random.default_rng(n + 1)
    x = rng.standard_normal(n)
    vals = rng.standard_normal(colidx.size) if values else np.ones(colidx.size)
    y = apply.spmv(torch.from_numpy(rowptr).cuda(), torch.from_numpy(colidx).cuda(),
                   torch.from_numpy(x).cuda(),
                   torch.from_numpy(vals).cuda() if values else None).cpu().numpy()
    A = sp.csr_matrix((vals, colidx, rowptr), shape=(n, n))
    absum = sp.csr_matrix((np.abs(vals), colidx, rowptr), shape=(n, n)) @ np.abs(x)
    L = np.diff(rowptr).astype(np.float64)
    assert np.all(np.abs(y - A @ x) <= 2 * L * 2.0**-53 * absum)


@pytest.mark.gpu
def test_gpu_spmv_special_values():
    """Infinities and NaN reach the rows that hold them and no other."""
    import torch
    from paper_1610_08128_amd import apply

    n = 5000
    rowptr, colidx = _blocks_of_rows(n, 3)
    rng = np.random.default_rng(4)
    x = rng.standard_normal(n)
    vals = rng.standard_normal(colidx.size)
    at = rng.integers(0, colidx.size, 40)
    vals[at] = np.where(np.arange(40) % 2, np.nan, np.inf)
    x[rng.integers(0, n, 5)] = np.nan
    bad = ~np.isfinite(vals) | ~np.isfinite(x[colidx])
    rows = np.repeat(np.arange(n), np.diff(rowptr))
    want = np.zeros(n, bool)
    want[rows[bad]] = True
    y = apply.spmv(torch.from_numpy(rowptr).cuda(), torch.from_numpy(colidx).cuda(),
                   torch.from_numpy(x).cuda(), torch.from_numpy(vals).cuda()).cpu().numpy()
    assert np.array_equal(~np.isfinite(y), want)


@pytest.mark.gpu
def test_gpu_spmv_past_the_buffers():
    """A row of more entries than a wave's 32-bit offsets cover, among short
    ones, and a vector of 2^29 entries and more.  Whole numbers, so that every
    sum is exact."""
    import torch
    from paper_1610_08128_amd import apply

    long = (1 << 28) + 77
    rowptr = torch.tensor([0, 20, 20 + long, 50 + long], dtype=torch.int32, device="cuda")
    colidx = torch.zeros(50 + long, dtype=torch.int32, device="cuda")
    colidx[:20] = 1
    colidx[-30:] = 2
    colidx[100:1100] = 2
    print(f"row of {long}", flush=True)
    y = apply.spmv(rowptr, colidx, torch.tensor([1.0, 3.0, 5.0], dtype=torch.float64,
                                                device="cuda"))
    assert y.tolist() == [60.0, long + 4000.0, 150.0]
    del colidx
    n = (1 << 29) + 3
    print(f"vector of {n}", flush=True)
    rowptr = torch.zeros(n + 1, dtype=torch.int32, device="cuda")
    rowptr[n - 4:] = torch.tensor([0, 20, 40, 140, 141], dtype=torch.int32, device="cuda")
    colidx = torch.arange(n - 141, n, dtype=torch.int32, device="cuda")
    x = torch.zeros(n, dtype=torch.float64, device="cuda")
    x[-141:] = torch.arange(141, dtype=torch.float64, device="cuda")
    y = apply.spmv(rowptr, colidx, x)
    assert y[-4:].tolist() == [190.0, 590.0, float(sum(range(40, 140))), 140.0]
    assert not bool(y[:-4].any())

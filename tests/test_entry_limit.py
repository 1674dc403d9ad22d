"""Matrices of nearly 2^31 entries, whose last rows' clamped entry indices
pass that number: the product, and the checks of a graph's and of a batch's
rows, which find the last entry and nothing behind it."""

import pytest

pytestmark = pytest.mark.gpu

ROW = 64


def _columns(n, nnz, local):
    """Column of entry e: e mod n, ascending in every row; the entries from
    `local` on, their own graph's, e - local mod 64."""
    import torch

    ci = torch.empty(nnz, dtype=torch.int32, device="cuda")
    step = 1 << 26
    for lo in range(0, nnz, step):
        e = torch.arange(lo, min(lo + step, nnz), device="cuda")
        ci[lo:lo + step] = torch.where(e < local, e % n, (e - local) % ROW).int()
    return ci


def _rowptr(n, nnz):
    import torch

    return torch.clamp(torch.arange(n + 1, device="cuda") * ROW, max=nnz).int()


@pytest.mark.parametrize("entries", [2**31 - 1, 2**31 - 63])
def test_product(entries):
    """Whole numbers, so that every sum is exact."""
    import torch
    from paper_1610_08128_amd import apply

    n = 1 << 25
    print(f"entries {entries}", flush=True)
    x = torch.randint(-1000, 1000, (n,), device="cuda").double()
    ci = _columns(n, entries, entries)
    y = apply.spmv(_rowptr(n, entries), ci, x)
    want = x.view(-1, ROW).sum(1).repeat(n * ROW // n)
    want[-1] -= x[ROW * (n - 1) % n:][entries - ROW * (n - 1):][:n * ROW - entries].sum()
    assert torch.equal(y, want)


@pytest.mark.parametrize("batch", [False, True])
def test_row_checks(batch):
    """Only the matrix's last entry is wrong: not a column, or another
    graph's."""
    import numpy as np
    import torch
    from paper_1610_08128_amd import rcm

    n, entries = 1 << 25, 2**31 - 2
    first = n - ROW
    print(f"entries {entries} batch {batch}", flush=True)
    ci = _columns(first if batch else n, entries, ROW * first if batch else entries)
    rp = _rowptr(n, entries)
    with pytest.raises(rcm.RcmError) as e:
        if batch:
            ci[-1] = -1  # the last vertex of the first graph
            rp = torch.cat([rp[:first + 1], rp[first:] - ROW * first])
            rcm.order_batched(np.array([0, first, n]), np.array([0, ROW * first, entries]), rp, ci)
        else:
            ci[-1] = n
            rcm.order(rp, ci)
    assert e.value.status == rcm.ERR_BAD_CSR

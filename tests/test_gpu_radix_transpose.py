"""The radix form of als_csr_to_csc, bit for bit against the oracle's stable transpose: one, two and
three passes (column counts around 256 and 65,536), entry counts around a tile (4,096) and a range,
rows of every length (empty runs, rows across tiles, one row, unsorted columns), columns without
entries, invalid columns, and a workspace too small for the sort, where the counting form runs."""
import numpy as np
import pytest
import torch

import oracle
from tests.gpu_util import log, to_dev

pytestmark = pytest.mark.gpu


def matrix(rng, m, n, nnz, shape):
    if shape == "one_row":
        counts = np.zeros(m, np.int64)
        counts[m // 2] = min(nnz, n)
    elif shape == "gaps":      # long runs of empty rows, then rows that start together
        counts = np.where(rng.random(m) < 0.05, rng.integers(1, max(2, n // 4), m), 0)
    else:
        counts = rng.multinomial(nnz, rng.dirichlet(np.ones(m))) if shape == "skewed" else \
            np.full(m, nnz // m)
    counts = np.minimum(counts, n).astype(np.int64)
    rowptr = np.zeros(m + 1, np.int64)
    rowptr[1:] = np.cumsum(counts)
    # distinct columns in a row, in no order: a stretch of a permutation, popular ones first
    place = rng.permutation(n).astype(np.int32)
    start = (rng.random(m) ** 3 * n).astype(np.int64)
    at = np.repeat(start - rowptr[:-1], counts) + np.arange(rowptr[-1])
    return rowptr, place[at % n], rng.standard_normal(int(rowptr[-1])).astype(np.float32)


def check(ctx, m, n, rowptr, colidx, vals):
    from paper_1603_03820_amd import als
    dev = ctx.device
    nnz = int(rowptr[-1])
    pad = max(nnz, 1)
    ci = np.zeros(pad, np.int32)
    ci[:nnz] = colidx
    vv = np.zeros(pad, np.float32)
    vv[:nnz] = vals
    out = (torch.full((n + 1,), -7, dtype=torch.int64, device=dev),
           torch.full((pad,), -7, dtype=torch.int32, device=dev),
           torch.full((pad,), -7.0, dtype=torch.float32, device=dev))
    cp, ri, vt = als.als_csr_to_csc(ctx, to_dev(rowptr, dev), to_dev(ci, dev), to_dev(vv, dev), m, n,
                                    nnz=nnz, out=out)
    torch.cuda.synchronize()
    valid = (colidx >= 0) & (colidx < n)
    rows = np.repeat(np.arange(m, dtype=np.int32), np.diff(rowptr))[valid]
    order = np.argsort(colidx[valid], kind="stable")
    k = len(order)
    assert np.array_equal(cp.cpu().numpy(),
                          np.concatenate([[0], np.cumsum(np.bincount(colidx[valid], minlength=n))]))
    assert np.array_equal(ri.cpu().numpy()[:k], rows[order])
    assert np.array_equal(vt.cpu().numpy()[:k].view(np.uint32), vals[valid][order].view(np.uint32))


def capacity(ctx, n):
    """Entries that the sort's part of the workspace holds (n > 256): what the status block, the scan's
    tile sums, the digit counts, the lower values' counts and starts and the arrays' alignment leave,
    at 10 bytes an entry up to 65,536 columns and 12 beyond."""
    def up(x):
        return (x + 255) // 256 * 256
    status = up(256 + 16 * 64 * 4)
    sums = up(8 * ((n + 4095) // 4096 + 1))
    counters = up(4 * 256 * 1536) + up(4 * 256) + up(4 << 16) + up(4 * ((1 << 16) + 1))
    return (ctx.workspace.numel() - status - sums - counters - 4 * 256) // (10 if n <= 65_536 else 12)


@pytest.mark.parametrize("n", [1, 255, 256, 257, 4000, 65_536, 65_537, 300_000])
@pytest.mark.parametrize("m,nnz,shape", [(1, 1, "even"), (700, 4_095, "even"), (700, 4_096, "skewed"),
                                         (700, 4_097, "skewed"), (3, 200_000, "one_row"),
                                         (20_000, 0, "gaps"), (5_000, 900_000, "skewed")])
def test_against_a_stable_sort(n, m, nnz, shape):
    from paper_1603_03820_amd import als
    rng = np.random.default_rng(n + m)
    if shape == "gaps" and n > 5_000:
        pytest.skip("rows of n / 4 entries: more than the case needs")
    rowptr, colidx, vals = matrix(rng, m, n, nnz, shape)
    log(f"radix transpose m={m} n={n} nnz={int(rowptr[-1])} {shape}")
    check(als.Context(0, 16), m, n, rowptr, colidx, vals)


@pytest.mark.parametrize("n", [200, 3_000, 70_000])
def test_invalid_columns_are_skipped(n):
    from paper_1603_03820_amd import als
    rng = np.random.default_rng(n)
    rowptr, colidx, vals = matrix(rng, 900, n, 60_000, "skewed")
    colidx = colidx.copy()
    colidx[rng.random(len(colidx)) < 0.1] = -1
    colidx[rng.random(len(colidx)) < 0.1] = n
    colidx[rng.random(len(colidx)) < 0.02] = 2 ** 31 - 1
    log(f"radix transpose, invalid columns, n={n}")
    check(als.Context(0, 16), 900, n, rowptr, colidx, vals)


def test_agrees_with_the_oracle(oracle_lib):
    """The numpy statement above is the oracle's transpose."""
    from paper_1603_03820_amd import als
    rng = np.random.default_rng(3)
    m, n = 3_000, 2_000
    rowptr, colidx, vals = matrix(rng, m, n, 150_000, "skewed")
    cp, ri, vt = oracle.get().transpose(rowptr, colidx, vals, m, n)
    ctx = als.Context(0, 16)
    got = als.als_csr_to_csc(ctx, *(to_dev(a, ctx.device) for a in (rowptr, colidx, vals)), m, n)
    for a, b in zip(got, (cp, ri, vt)):
        assert np.array_equal(a.cpu().numpy(), np.asarray(b))


@pytest.mark.parametrize("n", [3_000, 80_000])
@pytest.mark.parametrize("over", [0, 1, 100_000])
def test_both_sides_of_the_capacity(monkeypatch, n, over):
    """As many entries as the smallest workspace (f_max = 1, one wave per CU) holds, sorted in two and
    three passes in arrays that fill it, and more, which take the counting form."""
    from paper_1603_03820_amd import als
    monkeypatch.setenv("ALS_WAVES_PER_CU", "1")
    ctx = als.Context(0, 1)
    m, nnz = 6_000, capacity(ctx, n) + over
    rng = np.random.default_rng(n)
    counts = np.full(m, nnz // m) + (np.arange(m) < nnz % m)
    assert 100_000 < nnz <= m * n and counts.max() <= n
    rowptr = np.concatenate([[0], np.cumsum(counts)]).astype(np.int64)
    place = rng.permutation(n).astype(np.int32)
    start = (rng.random(m) ** 3 * n).astype(np.int64)
    at = np.repeat(start - rowptr[:-1], counts) + np.arange(nnz)
    log(f"radix transpose at its capacity n={n} nnz={nnz} workspace {ctx.workspace.numel()}")
    check(ctx, m, n, rowptr, place[at % n], rng.standard_normal(nnz).astype(np.float32))


@pytest.mark.parametrize("n", [200, 2_900])
def test_more_entries_than_the_matrix_has_places(monkeypatch, n):
    """The first n columns of a wider CSR: the entries outside [0, n) are skipped but count towards
    what the workspace holds, here more than it does although m n is not."""
    from paper_1603_03820_amd import als
    monkeypatch.setenv("ALS_WAVES_PER_CU", "1")
    ctx = als.Context(0, 1)
    rng = np.random.default_rng(n)
    m, wide = 100, 4_000
    rowptr = np.arange(m + 1, dtype=np.int64) * wide
    colidx = np.concatenate([rng.permutation(wide) for _ in range(m)]).astype(np.int32)
    vals = rng.standard_normal(m * wide).astype(np.float32)
    assert n <= 256 or m * n <= capacity(ctx, n) < m * wide   # (one pass has no limit)
    log(f"radix transpose, first {n} of {wide} columns, workspace {ctx.workspace.numel()}")
    check(ctx, m, n, rowptr, colidx, vals)

"""How the half-sweep's waves come by their chunks: short sweeps run fixed shares, longer ones claim
from striped counters.  Both sides of the line between them, against the fp64 oracle on every row
(the sums are the same fixed-order fp32 sums on both sides, so the bar is the parity bar, 1e-3, and
the observed error about 1e-6)."""
import numpy as np
import pytest
import torch

import oracle
from tests.gpu_util import gpu_half_sweep, log, row_rel_err

pytestmark = pytest.mark.gpu

# rank -> entry equivalents per wave up to which shares are fixed (fewer from four column blocks on)
STATIC_ENTRIES = {8: 2048, 47: 2048, 50: 512}


@pytest.mark.parametrize("f", sorted(STATIC_ENTRIES))
@pytest.mark.parametrize("over", [0, 1])
@pytest.mark.parametrize("waves_per_cu", [None, 1])
def test_fixed_shares_and_claims(monkeypatch, oracle_lib, f, over, waves_per_cu):
    from paper_1603_03820_amd import als
    if waves_per_cu:
        monkeypatch.setenv("ALS_WAVES_PER_CU", str(waves_per_cu))
    n, per_row = 300, 40
    ctx = als.Context(0, f)
    dummy = torch.zeros(2, dtype=torch.int64, device=ctx.device)
    _, (chunks, c_nnz, c_row, _, waves, _) = als.als_plan(ctx, dummy, 1, f)
    # the largest m whose cost is within the limit, or one row more
    m = STATIC_ENTRIES[f] * c_nnz * waves // (c_nnz * per_row + c_row) + over
    log(f"claims: W={waves} C={chunks} m={m} over={over}")
    rng = np.random.default_rng(7)
    rowptr = np.arange(m + 1, dtype=np.int64) * per_row
    start = rng.integers(0, n, size=m)
    colidx = np.sort((start[:, None] + 7 * np.arange(per_row)) % n, axis=1).astype(np.int32).ravel()
    vals = rng.uniform(1.0, 5.0, size=m * per_row).astype(np.float32)
    theta = rng.normal(0.2, 0.3, size=(n, f)).astype(np.float32)
    x = gpu_half_sweep(ctx, rowptr, colidx, vals, m, n, f, 0.05, theta)
    xo, _ = oracle.get().half_sweep(rowptr, colidx, vals, m, n, f, 0.05, theta.astype(np.float64))
    assert np.isfinite(x).all()
    assert row_rel_err(x, xo).max() <= 1e-3
    again = gpu_half_sweep(ctx, rowptr, colidx, vals, m, n, f, 0.05, theta)
    assert np.array_equal(x, again)


@pytest.mark.parametrize("f", [5, 40])
@pytest.mark.parametrize("lengths", [[3000] * 5, [4096, 4097, 4353, 12_000], [200_000, 257, 90_000],
                                     [383, 384, 385, 511, 512, 513, 640, 20, 0, 16_640]])
def test_cut_rows_of_a_short_sweep(oracle_lib, f, lengths):
    """Chunks smaller than the cut grid: hundreds of boundaries fall on a row's few cut points, in
    rows just short of and past the length from which pieces are summed in two passes (4,096)."""
    from paper_1603_03820_amd import als
    rng = np.random.default_rng(len(lengths))
    n = 250_000
    rowptr = np.zeros(len(lengths) + 1, np.int64)
    rowptr[1:] = np.cumsum(lengths)
    colidx = np.concatenate([np.sort(rng.choice(n, size=c, replace=False))
                             for c in lengths]).astype(np.int32)
    vals = rng.uniform(1.0, 5.0, size=int(rowptr[-1])).astype(np.float32)
    theta = rng.normal(0.1, 0.3, size=(n, f)).astype(np.float32)
    m = len(lengths)
    log(f"cut rows f={f} lengths={lengths}")
    ctx = als.Context(0, f)
    x = gpu_half_sweep(ctx, rowptr, colidx, vals, m, n, f, 0.05, theta)
    xo, _ = oracle.get().half_sweep(rowptr, colidx, vals, m, n, f, 0.05, theta.astype(np.float64))
    # fp32 sums of up to 200,000 terms, rounded once per 32: sqrt(6250) 2^-24 = 5e-6 of a Gram entry,
    # times a condition number below 30
    assert row_rel_err(x, xo).max() <= 1.5e-4
    assert np.array_equal(x, gpu_half_sweep(ctx, rowptr, colidx, vals, m, n, f, 0.05, theta))

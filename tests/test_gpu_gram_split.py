"""The Gram by bf16 part products: row lengths around the 32-entry group and the 64-entry index
batch, every form of the last block column (rating alone, packed, ordinary tiles) and both gather
forms, against the fp64 oracle; values near the top of the fp32 range; and the accuracy of long
and of cancelling sums against fp64.

Bars: the parts add up to the value exactly and the dropped products are below 2^-23 of a
product, so a Gram entry errs by less than the fp32 form's n rounding errors; with lambda n_u on the
diagonal the systems here have condition numbers below 1e3, so 1e3 x 2^-23 = 1.2e-4 bounds a row,
inside the parity bar of 1e-3; 2e-5 is asserted (measured: 3e-7 to 2e-6)."""
import os

import numpy as np
import pytest

import oracle
from tests.gpu_util import gpu_half_sweep, log, row_rel_err

pytestmark = pytest.mark.gpu

LENGTHS = [0, 1, 2, 3, 4, 5, 31, 32, 33, 63, 64, 65, 95, 96, 97, 127, 128, 129, 255, 257, 700]


def context(form, f):
    from paper_1603_03820_amd import als
    if form == "global":
        os.environ["ALS_GATHER"] = "global"
    try:
        return als.Context(0, f)
    finally:
        os.environ.pop("ALS_GATHER", None)


def rows(rng, n, lengths):
    rowptr = np.zeros(len(lengths) + 1, np.int64)
    rowptr[1:] = np.cumsum(lengths)
    colidx = np.concatenate([np.sort(rng.choice(n, size=c, replace=False)) for c in lengths])
    return rowptr, colidx.astype(np.int32)


@pytest.mark.parametrize("f", [1, 4, 11, 16, 20, 32, 36, 63, 100, 112, 115, 120, 128])
@pytest.mark.parametrize("form", ["buffer", "global"])
def test_group_edges(f, form):
    rng = np.random.default_rng(f)
    n = 800
    rowptr, colidx = rows(rng, n, LENGTHS * 3)
    m = len(rowptr) - 1
    vals = rng.uniform(1.0, 5.0, size=int(rowptr[-1])).astype(np.float32)
    theta = (rng.normal(size=(n, f)) * f ** -0.5 + 0.05).astype(np.float32)
    log(f"gram split f={f} form={form} rows={m}")
    x = gpu_half_sweep(context(form, f), rowptr, colidx, vals, m, n, f, 0.05, theta)
    xo, _ = oracle.get().half_sweep(rowptr, colidx, vals, m, n, f, 0.05, theta.astype(np.float64))
    assert np.all(x[np.diff(rowptr) == 0] == 0.0)
    assert row_rel_err(x, xo).max() <= 2e-5


@pytest.mark.parametrize("f", [4, 16, 21, 100])
def test_ratings_near_the_top_of_the_range(f):
    """b = sum r theta stays finite although r rounds up past the largest bf16 value."""
    rng = np.random.default_rng(f)
    n = 300
    rowptr, colidx = rows(rng, n, [1, 7, 33, 64])
    m = len(rowptr) - 1
    vals = np.full(int(rowptr[-1]), 3.4e38, np.float32)
    theta = (rng.normal(size=(n, f)) * 1e-4).astype(np.float32)
    log(f"gram split: ratings of 3.4e38, f={f}")
    x = gpu_half_sweep(context("buffer", f), rowptr, colidx, vals, m, n, f, 1.0, theta)
    xo, _ = oracle.get().half_sweep(rowptr, colidx, vals, m, n, f, 1.0, theta.astype(np.float64))
    assert np.isfinite(x).all()
    # one term alone is rounded once per operation; the longer sums cancel (random signs)
    assert row_rel_err(x, xo).max() <= 2e-5


@pytest.mark.parametrize("length", [40, 2_000, 60_000])
@pytest.mark.parametrize("mean", [0.0, 0.1])
def test_long_sums_keep_fp32_accuracy(length, mean):
    """A fp32 running sum of n products errs by about sqrt(n) 2^-25 of its value (more when every
    rounding goes one way); rounding an accumulator once per 32 entries must not do worse than
    that with a factor of 4 for the solve."""
    f, n = 36, 70_000
    rng = np.random.default_rng(length)
    rowptr, colidx = rows(rng, n, [length] * 4)
    vals = rng.normal(1.0, 1.0, size=4 * length).astype(np.float32)
    theta = rng.normal(mean, 0.1, size=(n, f)).astype(np.float32)
    log(f"gram split accuracy n={length} mean={mean}")
    x = gpu_half_sweep(context("buffer", f), rowptr, colidx, vals, 4, n, f, 0.05, theta)
    xo, _ = oracle.get().half_sweep(rowptr, colidx, vals, 4, n, f, 0.05, theta.astype(np.float64))
    # condition number of A: (f mean^2 + 0.01 + lambda) / (0.01 + lambda)
    cond = (f * mean ** 2 + 0.06) / 0.06
    bound = 4 * cond * max(4.0, length ** 0.5) * 2.0 ** -25
    err = float(np.linalg.norm(x - xo) / np.linalg.norm(xo))
    print(f"[gpu] relative error {err:.2e}, bound {bound:.2e}")
    assert err <= bound

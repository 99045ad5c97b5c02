"""The Gram by bf16 part products: row lengths around the 32-entry group and the 64-entry index
batch, every form of the last block column (rating alone, packed, ordinary tiles) and both gather
forms, against the fp64 oracle; values near the top of the fp32 range; the accuracy of long
and of cancelling sums against fp64; and the sums' own error beside that of fp32 products.

Bars: the parts add up to the value exactly and the dropped products are below 2^-22 of a
product; with lambda n_u on the diagonal the systems here have condition numbers below 1e3, so
1e3 x 2^-22 = 2.4e-4 bounds a row, inside the parity bar of 1e-3; 2e-5 is asserted (measured: 3e-7
to 2e-6)."""
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


def constants_with_large_parts(rng, shape):
    """Values h + m + l whose middle part is near its largest, 2^-7 of the leading bit, and whose low part
    is negative and near its largest, 2^-16: the products m l and l m, which the split form leaves
    out, are near 2^-23 each and have one sign."""
    h = 1.0 + rng.integers(0, 128, shape) / 128.0
    m = (128 + 8 * rng.integers(0, 16, shape) + 7) * 2.0 ** -15
    return (h + m - 0.9 * 2.0 ** -16).astype(np.float32)


@pytest.mark.parametrize("f", [4, 6, 16, 36, 63, 100, 115, 128])
@pytest.mark.parametrize("kind", ["random", "equal", "parts"])
@pytest.mark.parametrize("form", ["buffer", "global"])
def test_sums_err_no_more_than_fp32_products(f, kind, form):
    """The error of b = sum r theta against fp64, by itself: with lambda n = 2^40 the Gram matrix is
    below half a unit in the last place of the diagonal, every pivot is 2^40, and x = 2^-40 b without
    another rounding.  It must not exceed that of fp32 products summed one after the other, each
    entry an FMA (f a multiple of 16: four sums of every fourth entry, then their sum), neither at most
    nor as a root mean square (a tenth more is allowed: both are estimates from some thousand sums), at
    lengths on both sides of the shortest pieces' fp32 form (16 entries), where equal entries err
    most, and of the 32-entry group; one product alone is rounded to nearest exactly."""
    ctx = context(form, f)
    rng = np.random.default_rng(f)
    for length in (1, 2, 3, 8, 15, 16, 17, 20, 31, 32, 33, 64, 128):
        m = max(64, 4096 // length)
        shape = (m, length, f) if kind == "random" else (m, 1, f)
        if kind == "parts":
            theta = constants_with_large_parts(rng, shape)
            vals = constants_with_large_parts(rng, shape[:2])
        else:
            theta = rng.uniform(0.5, 1.5, shape).astype(np.float32)
            vals = rng.uniform(1.0, 5.0, shape[:2]).astype(np.float32)
        theta = np.broadcast_to(theta, (m, length, f)).reshape(m * length, f).copy()
        vals = np.broadcast_to(vals, (m, length)).reshape(-1).copy()
        rowptr = np.arange(m + 1, dtype=np.int64) * length
        log(f"gram split, sums of {length}, {kind}, f={f} {form}")
        lam = 2.0 ** 40 / length
        assert np.float32(np.float64(np.float32(lam)) * length) == np.float32(2.0 ** 40)
        x = gpu_half_sweep(ctx, rowptr, np.arange(m * length, dtype=np.int32), vals, m, m * length, f,
                           lam, theta)
        got = x.astype(np.float64) * 2.0 ** 40
        products = (vals[:, None].astype(np.float64) * theta).reshape(m, length, f)
        slots = 4 if f % 16 == 0 else 1
        chains = np.zeros((slots, m, f), np.float32)
        for k in range(length):
            at = k % slots
            chains[at] = (chains[at].astype(np.float64) + products[:, k]).astype(np.float32)
        chain = chains[0]
        for other in chains[1:]:
            chain = chain + other
        b = products.sum(1)
        err, ref = np.abs(got / b - 1.0), np.abs(chain / b - 1.0)
        print(f"[gpu] max {err.max():.2e} chain {ref.max():.2e}; rms {np.sqrt((err ** 2).mean()):.2e} "
              f"chain {np.sqrt((ref ** 2).mean()):.2e}")
        if length == 1:
            assert np.array_equal(got, chain.astype(np.float64))
        assert err.max() <= 1.1 * ref.max()
        assert (err ** 2).mean() <= 1.21 * (ref ** 2).mean()


@pytest.mark.parametrize("f", [6, 16, 20, 63, 100, 115, 128])
@pytest.mark.parametrize("exponent", [-105, -115, -122])
@pytest.mark.parametrize("what", ["ratings", "theta", "column", "zeros"])
def test_tiny_values_keep_their_bits(f, exponent, what):
    """bf16's smallest numbers are fp32's, but not its subnormals, so the parts of values below about
    2^-110 lose bits; rows whose ratings, or a whole column of whose factors, are that small are summed
    with fp32 products.  Whole rows and rows cut between chunks (30,000 entries), scaled by a power of
    two: x_u (of "column": its entry for the column) agrees with fp64 as it does unscaled (twice that
    error and 2e-5, plus what results that small lose to fp32's own subnormals)."""
    rng = np.random.default_rng(f - exponent)
    n = 40_000
    rowptr, colidx = rows(rng, n, [3, 17, 40, 64, 200, 1_500, 30_000, 33, 30_000, 16])
    m = len(rowptr) - 1
    vals = rng.uniform(1.0, 5.0, size=int(rowptr[-1])).astype(np.float32)
    theta = (rng.normal(size=(n, f)) * f ** -0.5 + 0.05).astype(np.float32)
    plain = vals.copy(), theta.copy()
    scale = np.float32(2.0 ** exponent)
    if what == "ratings":
        vals *= scale
    elif what == "theta":
        theta *= scale
    elif what == "column":
        theta[:, f // 2] *= scale
    else:   # a column and a row's ratings of zeros
        theta[:, f // 2] = 0.0
        vals[rowptr[3]:rowptr[4]] = 0.0
    log(f"gram split, tiny {what}, 2^{exponent}, f={f}")

    def both(vals, theta):
        xo, _ = oracle.get().half_sweep(rowptr, colidx, vals, m, n, f, 0.05, theta.astype(np.float64))
        return [gpu_half_sweep(context(form, f), rowptr, colidx, vals, m, n, f, 0.05, theta)
                for form in ("buffer", "global")], xo

    bar = row_rel_err(*(a if i else a[0] for i, a in enumerate(both(*plain)))).max() * 2 + 2e-5
    results, xo = both(vals, theta)
    for x in results:
        assert np.isfinite(x).all()
        if what == "column":
            # its other entries as ever; the entry is a difference of sums of its size, so a cancellation
            # down to a tenth is allowed for
            assert row_rel_err(np.delete(x, f // 2, 1), np.delete(xo, f // 2, 1)).max() <= bar
            got, ref = x[:, f // 2].astype(np.float64), xo[:, f // 2]
            assert np.abs(got - ref).max() <= 10 * bar * np.abs(ref).max() + f * 2.0 ** -146
        elif what == "zeros":
            assert np.all(x[:, f // 2] == 0.0) and np.all(x[3] == 0.0)
            assert row_rel_err(np.delete(x, 3, 0), np.delete(xo, 3, 0)).max() <= bar
        else:
            err = np.abs(x.astype(np.float64) - xo).max(axis=1)
            assert np.all(err <= bar * np.abs(xo).max(axis=1) + f * 2.0 ** -146)

"""MCC of few input channels on three-slice values: edges of its blocks, chunks and channel slices, and the values the
slices do not carry, against double precision."""
import numpy as np
import pytest

import paper_2405_05118_amd as mdh
from paper_2405_05118_amd import binding as B

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def reference(x, f, st):
    N, H, W, C = x.shape
    K, R, S, _ = f.shape
    P, Q = (H - R) // st + 1, (W - S) // st + 1
    x, f = x.astype(np.float64), f.astype(np.float64)
    out = np.zeros((N, P, Q, K))
    with np.errstate(invalid="ignore"):
        for r in range(R):
            for s in range(S):
                tap = x[:, r : r + (P - 1) * st + 1 : st, s : s + (Q - 1) * st + 1 : st, None, :]
                out += (tap * f[None, None, None, :, r, s, :]).sum(axis=-1)
    return out


def run(x, f, st, params=None):
    N, H, W, C = x.shape
    K, R, S, _ = f.shape
    P, Q = (H - R) // st + 1, (W - S) // st + 1
    if params is None:  # a call without a table is the kernel that this file is about
        p = mdh.mdh_call_params(mdh.MDH_MCC, (N, P, Q, K, C, R, S, st, st))
        assert p.blk[4] == 1 and p.in_region[0] == B.MR_HBM
    out = torch.full((N * P * Q * K + 64,), -7.0, device="cuda")  # guard words behind the output
    mdh.mdh_mcc(torch.from_numpy(x).cuda(), torch.from_numpy(f).cuda(), out[: N * P * Q * K].view(N, P, Q, K), (st, st), params, None)
    assert (out[N * P * Q * K :] == -7.0).all()
    return out[: N * P * Q * K].view(N, P, Q, K).cpu().numpy()


def close(got, want, terms):
    # four times the error fp32 sums of random products show against 64 bits, 1.8e-8 sqrt(terms), 1.2e-7 at the least: a
    # product of slices left out shows as 1e-6 or more
    assert np.linalg.norm(got - want) <= max(5e-7, 7.2e-8 * np.sqrt(terms)) * np.linalg.norm(want)


def data(N, H, W, C, K, R, S):
    rng = np.random.default_rng(N + 3 * H + 5 * W + 7 * C + 11 * K)
    return rng.standard_normal((N, H, W, C)).astype(np.float32), rng.standard_normal((K, R, S, C)).astype(np.float32)


# outputs of one block and less, one row or column more; an odd and an even number of chunks, a last chunk of one value and
# a full one; channels below, at and above a slice of 32 and of 64; an input that ends inside a 16-byte load
SHAPES = [(1, 7, 7, 3, 1, 7, 7, 1), (1, 8, 22, 3, 31, 7, 7, 1), (2, 9, 39, 3, 33, 7, 7, 1), (1, 22, 23, 2, 64, 7, 7, 2),
          (3, 20, 21, 4, 65, 5, 5, 2), (1, 21, 37, 8, 40, 3, 3, 1), (2, 33, 18, 5, 16, 3, 5, 1), (1, 70, 70, 1, 7, 7, 7, 3),
          (1, 9, 64, 3, 8, 3, 3, 1), (2, 11, 12, 6, 96, 5, 7, 1), (1, 5, 5, 7, 3, 5, 5, 1), (1, 3, 300, 3, 5, 3, 3, 1)]


@pytest.mark.parametrize("shape", SHAPES + [(40, 64, 70, 3, 64, 5, 5, 1), (36, 70, 72, 2, 130, 7, 7, 1)])
def test_against_double(shape):
    *d, st = shape
    x, f = data(*d)
    close(run(x, f, st), reference(x, f, st), f[0].size)


# an infinity, a NaN, an overflow: exactly the outputs whose windows hold it, also beside a window's last value
@pytest.mark.parametrize("shape", [(1, 30, 41, 3, 33, 7, 7, 1), (2, 23, 23, 3, 64, 7, 7, 2), (1, 19, 40, 4, 5, 3, 3, 1)])
@pytest.mark.parametrize("value", [np.inf, np.nan, 3e38])
def test_values_out_of_range(shape, value):
    *d, st = shape
    x, f = data(*d)
    x[0, 7, 8, 0], x[0, 0, 11, -1], x[-1, -1, -1, -1] = value, -value, value
    if value == 3e38:
        f[f.shape[0] // 2] *= 8
    want, got = reference(x, f, st), run(x, f, st)
    with np.errstate(over="ignore"):
        want32 = want.astype(np.float32)
    odd = ~np.isfinite(want32)
    assert np.array_equal(np.isnan(want32), np.isnan(got)) if value != 3e38 else True
    assert not np.isfinite(got[odd]).any() and np.isfinite(got[~odd]).all()
    assert np.array_equal(got[np.isinf(want32)], want32[np.isinf(want32)]) if value != 3e38 else True
    low = np.abs(want) < 1e30
    close(got[low], want[low], f[0].size)


# magnitudes whose last slices would be lost, in the input, in the filter, in one channel or pixel beside ordinary ones
@pytest.mark.parametrize("where", ["input", "filter", "channel", "pixels"])
def test_small_magnitudes(where):
    x, f = data(1, 30, 41, 3, 40, 7, 7)
    tiny = np.float32(2.0**-112)
    if where == "input":
        x *= tiny
    elif where == "filter":
        f *= tiny
    elif where == "channel":
        f[3] *= tiny
    else:
        x[:, 10:20, 10:20] *= tiny
    want, got = reference(x, f, 1), run(x, f, 1)
    close(got, want, f[0].size)
    if where == "channel":
        close(got[..., 3], want[..., 3], f[0].size)
    if where == "pixels":
        close(got[:, 10:14, 10:14], want[:, 10:14, 10:14], f[0].size)


# The row below the last windows is in none of them, whatever it holds: with an even number of chunks it is what a next step
# would take.  The filter's middle slices would be lost to subnormal numbers.
@pytest.mark.parametrize("value", [np.inf, np.nan, 3e38])
def test_what_lies_below_the_windows(value):
    x, f = data(1, 8, 40, 2, 33, 7, 7)
    f *= np.float32(2.0**-118)
    x[0, 7] = value
    close(run(x, f, 2), reference(x, f, 2), f[0].size)


# zeros are exact, and cost no second evaluation's rounding: a dead filter, a blank patch, a delta filter
def test_zeros_and_single_products():
    x, f = data(2, 40, 41, 3, 40, 7, 7)
    x[0, 5:30, 5:30] = 0
    f[7] = 0
    f[9] = 0
    f[9, 2, 3, 1] = 1
    got = run(x, f, 1)
    assert (got[..., 7] == 0).all() and (got[0, 5:24, 5:24] == 0).all()
    assert np.array_equal(got[..., 9], x[:, 2 : 2 + 34, 3 : 3 + 35, 1])


# its tables are candidates, behind those of the fp32 instructions, and what a call without a table runs is one of them
def test_tables():
    x, f = data(2, 40, 43, 3, 64, 7, 7)
    s = (2, 34, 37, 64, 3, 7, 7, 1, 1)
    tables = [mdh.mdh_candidate(mdh.MDH_MCC, s, i) for i in range(mdh.mdh_num_candidates(mdh.MDH_MCC, s))]
    split = [p for p in tables if p.blk[4] == 1 and p.in_region[0] == B.MR_HBM]
    assert len(split) == 6
    got, want = [run(x, f, 1, p) for p in split], reference(x, f, 1)
    for g in got:
        close(g, want, f[0].size)
    assert any(np.array_equal(g, run(x, f, 1)) for g in got)
    assert np.array_equal(run(x, f, 1, mdh.mdh_call_params(mdh.MDH_MCC, s)), run(x, f, 1))


def rel(got, want):
    return np.linalg.norm(got - want) / np.linalg.norm(want)


def both_tables(x, f):
    """The tables with fp32 instructions and with slices that a call is given first."""
    (N, H, W, C), (K, R, S, _) = x.shape, f.shape
    s = (N, H - R + 1, W - S + 1, K, C, R, S, 1, 1)
    few = [p for p in (mdh.mdh_candidate(mdh.MDH_MCC, s, i) for i in range(mdh.mdh_num_candidates(mdh.MDH_MCC, s))) if p.blk[4] == 1]
    return [p for p in few if p.in_region[0] != B.MR_HBM][0], [p for p in few if p.in_region[0] == B.MR_HBM]


# Sums of few terms: filters with n taps that are not zero, anywhere, one step after the other (16 values) or side by side,
# and inputs with few values that are not zero.  A step rounds a sum at most once, and the sum of all smaller products once
# more, so n terms are rounded no more often than by n multiply-adds; 4 % is what 10^5 outputs leave open (one term: the same
# error, but for a sum that lies within 2^-8 of a tie).
@pytest.mark.parametrize("where", ["anywhere", "steps", "together", "input"])
@pytest.mark.parametrize("terms", [1, 2, 3, 6, 17, 40])
def test_sums_of_few_terms(where, terms):
    rng = np.random.default_rng(terms)
    x, f = data(2, 38, 41, 3, 64, 7, 7)
    if where == "input":
        x = np.where(rng.random(x.shape) < terms / f[0].size, x, np.float32(0))
    else:
        n = f[0].size
        for k in range(len(f)):
            at = {"anywhere": rng.permutation(n)[:terms], "steps": (np.arange(terms) * 16 + rng.integers(n)) % n,
                  "together": (np.arange(terms) + rng.integers(n)) % n}[where]
            keep = np.zeros(n, bool)
            keep[at] = True
            f[k] = np.where(keep.reshape(f[k].shape), f[k], np.float32(0))
    want = reference(x, f, 1)
    fp32, split = both_tables(x, f)
    limit = 1.04 * rel(run(x, f, 1, fp32), want)
    for p in split + [None]:
        assert rel(run(x, f, 1, p), want) <= limit


# a filter of one tap: the product, rounded once, after a sum of the smaller products that is rounded 2^-8 as finely
def test_one_tap():
    x, f = data(2, 40, 41, 3, 40, 7, 7)
    f[:] = 0
    rng = np.random.default_rng(3)
    taps = [(int(rng.integers(7)), int(rng.integers(7)), int(rng.integers(3))) for _ in f]
    for k, t in enumerate(taps):
        f[(k,) + t] = np.float32(0.3) if k == 0 else np.float32(rng.standard_normal())
    got = run(x, f, 1)
    for k, (r, s, c) in enumerate(taps):
        want = x[:, r : r + 34, s : s + 35, c].astype(np.float64) * np.float64(f[k, r, s, c])
        assert (np.abs(got[..., k] - want) <= 2.0**-24 * (1 + 2.0**-7) * np.abs(want)).all(), k

"""Inf, NaN, overflow and values below 2^-100 through every view, part and tap of the kernels that carry a value as three
bf16 values: what such a value enters is what the fp32 instructions give, and so is all the rest."""
import pytest

import paper_2405_05118_amd as mdh
from test_split_products import split_candidates
from test_split_exact import workspace

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

INF, NAN, BIG = float("inf"), float("nan"), torch.finfo(torch.float32).max


def check(got, ref, mag, terms, what):
    """ref: the same sums in 64 bits.  Not finite in the same places (an output beyond the largest float is Inf), the
    others as exact as an fp32 sum of these terms, or as the subnormal numbers allow."""
    want = ref.float()
    assert torch.equal(torch.isnan(got), torch.isnan(want)), what
    assert torch.equal(got[torch.isinf(want)], want[torch.isinf(want)]), what
    fin = torch.isfinite(want)
    assert bool(torch.isfinite(got[fin]).all()), what
    assert bool(((got[fin].double() - ref[fin]).abs() <= terms * 2.0**-24 * mag[fin] + terms * 2.0**-149).all()), what


def sums(a, b):
    """a b and |a| |b| in 64 bits; 0 * Inf is NaN there too."""
    return a.double() @ b.double(), a.double().abs() @ b.double().abs()


# rows, columns and k of the special values: tile edges, both sides of where two and four parts of k meet, the tail
def plant(a, b, what, K):
    ks = (0, K // 4 - 1, K // 4, K // 2 - 1, K // 2, K - 2, K - 1)
    if what == "inf":
        for i, k in enumerate(ks):
            a[17 * i, k] = INF if i % 2 else -INF
        b[K - 1, 60], b[0, 3] = INF, 0.0
    elif what == "nan":
        a[63, K - 1], a[64, 0], b[K // 2, 33] = NAN, NAN, NAN
    elif what == "all nan":
        a[:] = NAN
    elif what == "overflow":
        a[31] = 0.0
        a[31, :2], b[1] = BIG, b[0]  # two equal products: beyond the largest float together, in any order, or not at all
    elif what == "tiny":
        a[65] *= 1e-38
        a[1] = 0.0
        a[1, K - 1] = 1e-42
        b[:, 2] = 0.0
        b[K // 2, 2] = 3e-39
        b[:, 5:] *= 1e20
    elif what == "underflow":  # products of slices below the smallest normal number
        a *= 1e-18
        b *= 1e-18


WHAT = ["inf", "nan", "all nan", "overflow", "tiny", "underflow"]


@pytest.mark.parametrize("what", WHAT)
@pytest.mark.parametrize("views", [None, (0, 0, 0), (1, 0, 0), (0, 1, 0), (1, 1, 0), (0, 0, 1), (1, 0, 1), (1, 1, 1)])
def test_special_values_in_products(what, views):
    M, N, K = 150, 130, 535  # tails of k-tiles of 16 and 32, parts of two and four
    ta, tb, tc = views or (0, 0, 0)
    batch = 1 if views is None else 2
    inst, sizes = (mdh.MDH_MATMUL, (M, N, K)) if views is None else (mdh.MDH_BMATMUL, (batch, M, N, K, ta, tb, tc))
    g = torch.Generator(device="cuda").manual_seed(len(what))
    a = torch.rand((batch, M, K), generator=g, device="cuda") * 2 - 1
    b = torch.rand((batch, K, N), generator=g, device="cuda") * 2 - 1
    plant(a[batch - 1], b[batch - 1], what, K)  # the last entry of a batch: the ones before it stay as they are
    refs = [sums(a[i], b[i]) for i in range(batch)]
    A, B = (a.transpose(1, 2).contiguous() if ta else a), (b.transpose(1, 2).contiguous() if tb else b)
    cands = split_candidates(inst, sizes, 2 if views is None else 3)
    kdim = 2 if views is None else 3
    assert {1, 2, 4} == {p.prt[3][kdim] for p in cands}
    for p in cands:
        C = torch.full((batch, N, M) if tc else (batch, M, N), 7.0, device="cuda")
        if views is None:
            mdh.mdh_matmul(A[0], B[0], C[0], p, workspace(inst, sizes, p))
        else:
            mdh.mdh_matmul_ex(A, B, C, bool(ta), bool(tb), bool(tc), p, workspace(inst, sizes, p))
        for i in range(batch):
            check(C[i].t() if tc else C[i], *refs[i], K, (p.table(), i))


# more blocks than the wavefronts of a 256-wide tile take one by one, and a row and a column of them
@pytest.mark.parametrize("what", ["inf", "all nan", "rows"])
def test_special_values_in_large_tiles(what):
    M, N, K = 600, 530, 333
    g = torch.Generator(device="cuda").manual_seed(5)
    a = torch.rand((M, K), generator=g, device="cuda") * 2 - 1
    b = torch.rand((K, N), generator=g, device="cuda") * 2 - 1
    if what == "rows":
        a[::90, 100] = INF
        b[7, 300:310] = NAN
    else:
        plant(a, b, what, K)
    ref = sums(a, b)
    for p in split_candidates(mdh.MDH_MATMUL, (M, N, K), 2):
        C = torch.full((M, N), 7.0, device="cuda")
        mdh.mdh_matmul(a, b, C, p, workspace(mdh.MDH_MATMUL, (M, N, K), p))
        check(C, *ref, K, p.table())


@pytest.mark.parametrize("what", WHAT)
@pytest.mark.parametrize("shape", [(2, 13, 37, 70, 131, 3, 3, 1), (1, 21, 40, 45, 70, 3, 2, 2), (1, 9, 33, 260, 40, 1, 1, 1)])
def test_special_values_in_convolutions(what, shape):
    N, H, W, C, K, R, S, st = shape
    P, Q = (H - R) // st + 1, (W - S) // st + 1
    g = torch.Generator(device="cuda").manual_seed(len(what) + C)
    x = torch.randn((N, H, W, C), generator=g, device="cuda")
    f = torch.randn((K, R, S, C), generator=g, device="cuda")
    if what == "inf":
        x[0, 5, 8, C - 1], x[N - 1, H - 1, W - 1, 0], f[33, R - 1, 0, C // 2] = INF, -INF, INF
    elif what == "nan":
        x[0, 0, 0, 3], f[K - 1, 0, S - 1, C - 1] = NAN, NAN
    elif what == "all nan":
        x[:] = NAN
    elif what == "overflow":
        x[0, 4, 4, :2] = BIG
        f[..., 0].clamp_(-0.9, 0.9)
        f[..., 1] = f[..., 0]
    elif what == "tiny":
        x[0, 3:8, 3:12] *= 1e-38
        f[2] = 0.0
        f[2, 0, 0, C - 1] = 1e-41
        x[:, :, 20:] *= 1e20
    else:
        x, f = x * 1e-18, f * 1e-18
    # windows by copying, so that a special value reaches its own windows alone
    win = x.double().unfold(1, R, st).unfold(2, S, st).permute(0, 1, 2, 4, 5, 3).reshape(N * P * Q, R * S * C)
    ref, mag = (t.view(N, P, Q, K) for t in sums(win, f.reshape(K, R * S * C).t().contiguous()))
    sizes = (N, P, Q, K, C, R, S, st, st)
    cands = split_candidates(mdh.MDH_MCC, sizes, 4)
    assert len({p.prt[3][4] for p in cands}) > 1  # one part of c and more
    for p in cands:
        out = torch.full((N, P, Q, K), 7.0, device="cuda")
        mdh.mdh_mcc(x, f, out, (st, st), p, workspace(mdh.MDH_MCC, sizes, p))
        check(out, ref, mag, R * S * C, p.table())

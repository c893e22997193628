"""Outputs that are zero because a row, a column, a filter or a window of pixels is: the kernels that carry a value as
three bf16 values tell them from outputs that underflow, and evaluate only the latter with fp32 instructions."""
import pytest

import paper_2405_05118_amd as mdh
from test_split_exact import tables, workspace

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def check(got, ref, mag, terms, what):
    assert bool((got[ref == 0] == 0).all()), what
    assert bool(((got.double() - ref).abs() <= terms * 2.0**-24 * mag + terms * 2.0**-149).all()), what


# zero rows and columns alone, with elements too small to split in a row of its own, in a zero row's tile, and in one
# that is zero but for them; K leaves a tail
@pytest.mark.parametrize("views", [None, (1, 0, 0), (0, 1, 0), (1, 1, 1)])
@pytest.mark.parametrize("tiny", ["none", "row", "in a zero row", "in a zero column"])
def test_zero_rows_and_columns(views, tiny):
    M, N, K = 700, 900, 700
    ta, tb, tc = views or (0, 0, 0)
    inst, sizes = (mdh.MDH_MATMUL, (M, N, K)) if views is None else (mdh.MDH_BMATMUL, (1, M, N, K, ta, tb, tc))
    g = torch.Generator(device="cuda").manual_seed(K)
    a = torch.rand((M, K), generator=g, device="cuda") * 2 - 1
    b = torch.rand((K, N), generator=g, device="cuda") * 2e6 - 1e6
    a[40:100] = 0.0
    a[M - 1] = 0.0
    b[:, 7] = 0.0
    b[:, 130:200] = 0.0
    if tiny == "row":
        a[5] *= 1e-38
    elif tiny == "in a zero row":
        a[41, K - 1] = 3e-39
    elif tiny == "in a zero column":
        b[0, 150] = -2e-41
    ref, mag = a.double() @ b.double(), a.double().abs() @ b.double().abs()
    A, B = (a.t().contiguous() if ta else a), (b.t().contiguous() if tb else b)
    for p in tables(inst, sizes):
        C = torch.full((N, M) if tc else (M, N), float("nan"), device="cuda")
        if views is None:
            mdh.mdh_matmul(A, B, C, p, workspace(inst, sizes, p))
        else:
            mdh.mdh_matmul_ex(A[None], B[None], C[None], bool(ta), bool(tb), bool(tc), p, workspace(inst, sizes, p))
        check(C.t() if tc else C, ref, mag, K, p and p.table())


# a dead filter, windows of zero pixels that end inside a tile, the same with one element too small to split
@pytest.mark.parametrize("shape", [(2, 24, 42, 70, 96, 3, 3, 1), (1, 30, 35, 200, 130, 1, 1, 1), (1, 37, 49, 48, 70, 5, 3, 2)])
@pytest.mark.parametrize("tiny", ["none", "pixel", "filter"])
def test_zero_pixels_and_filters(shape, tiny):
    N, H, W, C, K, R, S, st = shape
    P, Q = (H - R) // st + 1, (W - S) // st + 1
    g = torch.Generator(device="cuda").manual_seed(C)
    x = torch.randn((N, H, W, C), generator=g, device="cuda").clamp_(min=0)
    f = torch.randn((K, R, S, C), generator=g, device="cuda") * 1e6
    x[:, 10:20, 5:, :] = 0.0
    f[3], f[K - 1] = 0.0, 0.0
    if tiny == "pixel":
        x[0, 15, 20, C - 1] = 2e-39
    elif tiny == "filter":
        f[3, R - 1, 0, 0] = 1e-40
    win = x.double().unfold(1, R, st).unfold(2, S, st).permute(0, 1, 2, 4, 5, 3).reshape(N * P * Q, R * S * C)
    flat = f.double().reshape(K, R * S * C).t().contiguous()
    ref, mag = (win @ flat).view(N, P, Q, K), (win.abs() @ flat.abs()).view(N, P, Q, K)
    sizes = (N, P, Q, K, C, R, S, st, st)
    for p in tables(mdh.MDH_MCC, sizes):
        out = torch.full((N, P, Q, K), float("nan"), device="cuda")
        mdh.mdh_mcc(x, f, out, (st, st), p, workspace(mdh.MDH_MCC, sizes, p))
        check(out, ref, mag, R * S * C, p and p.table())


# Outputs that cancel to zero, in few rows and in more than are looked at one by one, with an element too small to split
# in the same row: what it adds is the result, to the accuracy of one product.
@pytest.mark.parametrize("views", [None, (1, 0, 0), (0, 1, 0), (1, 1, 1)])
@pytest.mark.parametrize("rows", [1, 40])
def test_cancelled_rows(views, rows):
    M, N, K = 700, 900, 700
    ta, tb, tc = views or (0, 0, 0)
    inst, sizes = (mdh.MDH_MATMUL, (M, N, K)) if views is None else (mdh.MDH_BMATMUL, (1, M, N, K, ta, tb, tc))
    g = torch.Generator(device="cuda").manual_seed(rows)
    a = torch.rand((M, K), generator=g, device="cuda") * 2 - 1
    b = torch.rand((K, N), generator=g, device="cuda") * 2e6 - 1e6
    a[300 : 300 + rows] = 0.0
    a[300 : 300 + rows, K - 3 :] = torch.tensor([1.0, -1.0, 3e-39])
    b[K - 2, 11], b[K - 1, 11] = b[K - 3, 11], 8e5
    b[K - 2, N - 1], b[K - 1, N - 1] = b[K - 3, N - 1], 0.0  # cancels and stays zero
    ref, mag = a.double() @ b.double(), a.double().abs() @ b.double().abs()
    A, B = (a.t().contiguous() if ta else a), (b.t().contiguous() if tb else b)
    for p in tables(inst, sizes):
        C = torch.full((N, M) if tc else (M, N), float("nan"), device="cuda")
        if views is None:
            mdh.mdh_matmul(A, B, C, p, workspace(inst, sizes, p))
        else:
            mdh.mdh_matmul_ex(A[None], B[None], C[None], bool(ta), bool(tb), bool(tc), p, workspace(inst, sizes, p))
        got = C.t() if tc else C
        check(got, ref, mag, K, p and p.table())
        # (a part boundary between the three leaves two sums of 1e6 that cancel when they are added: nothing lost either)
        want = ref[300 : 300 + rows, 11]
        assert bool(((got[300 : 300 + rows, 11].double() - want).abs() <= 1e-6 * want.abs()).all()), p and p.table()


@pytest.mark.parametrize("shape", [(2, 24, 42, 70, 96, 3, 3, 1), (1, 30, 35, 200, 130, 1, 1, 1), (1, 37, 49, 48, 70, 5, 3, 2)])
@pytest.mark.parametrize("pixels, filters", [(1, 1), (20, 1), (1, 30)])
def test_cancelled_pixels(shape, pixels, filters):
    N, H, W, C, K, R, S, st = shape
    P, Q = (H - R) // st + 1, (W - S) // st + 1
    g = torch.Generator(device="cuda").manual_seed(C)
    x = torch.randn((N, H, W, C), generator=g, device="cuda")
    f = torch.randn((K, R, S, C), generator=g, device="cuda") * 1e6
    x[:, 8:22, 3:35, :] = 0.0
    x[0, 12, 10 : 10 + pixels, :3] = torch.tensor([1.0, 1.0, 2e-40])
    f[5 : 5 + filters, ..., 1] = -f[5 : 5 + filters, ..., 0]
    f[5 : 5 + filters, ..., 2] = 1e6
    def sums(x):
        win = x.double().unfold(1, R, st).unfold(2, S, st).permute(0, 1, 2, 4, 5, 3).reshape(N * P * Q, R * S * C)
        flat = f.double().reshape(K, R * S * C).t().contiguous()
        return (win @ flat).view(N, P, Q, K), (win.abs() @ flat.abs()).view(N, P, Q, K)

    ref, mag = sums(x)
    # windows of which nothing but the planted pixels is not zero: the first two channels cancel, the third is the result
    inside = torch.zeros((P, Q), dtype=torch.bool, device="cuda")
    for p in range(P):
        for q in range(Q):
            inside[p, q] = 8 <= p * st and p * st + R <= 22 and 3 <= q * st and q * st + S <= 35
    third = x.clone()
    third[0, 12, 10 : 10 + pixels, :2] = 0.0
    where = torch.zeros_like(ref, dtype=torch.bool)
    where[0, ..., 5 : 5 + filters] = inside[..., None]
    ref = torch.where(where, sums(third)[0], ref)
    want = ref[where]
    assert bool((want.abs() > 0).any()) and float(want.abs().max()) < 1e-30
    sizes = (N, P, Q, K, C, R, S, st, st)
    for p in tables(mdh.MDH_MCC, sizes):
        out = torch.full((N, P, Q, K), float("nan"), device="cuda")
        mdh.mdh_mcc(x, f, out, (st, st), p, workspace(mdh.MDH_MCC, sizes, p))
        check(out, ref, mag, R * S * C, p and p.table())
        if pixels == 1 or R * S == 1:  # (two planted pixels in a window: what the first adds is lost against the second's 1e6)
            assert bool(((out[where].double() - want).abs() <= 1e-5 * want.abs()).all()), p and p.table()

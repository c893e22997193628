"""Dense sums through the kernels that carry an fp32 value as three bf16 values: accuracy of fp32, by a limit that any one
of the six products missing, in all of a result, exceeds.

The limit is a relative 2-norm: 1.8e-8 sqrt(terms) is what fp32 sums of products show (1.2e-7 at the least), three times
that is allowed.  A missing product with a low slice costs 4e-7 to 1e-6 whatever the number of terms, so the limit can tell
up to about 100 terms; in longer sums the exact sums of one term (test_split_exact) do, term by term.
"""
import math

import pytest

import paper_2405_05118_amd as mdh
from test_split_exact import workspace
from test_split_products import split_candidates

torch = pytest.importorskip("torch")

PRODUCTS = ("hh", "hm", "mh", "mm", "hl", "lh")


def limit(terms):
    return 3 * max(1.2e-7, 1.8e-8 * math.sqrt(terms))


def rel(got, ref):
    return float((got.double() - ref).norm() / ref.norm())


def slices(x):
    out = {}
    for name in "hml":
        out[name] = x.to(torch.bfloat16).float()
        x = x - out[name]
    assert bool((x == 0).all())  # three slices are the value
    return {k: v.double() for k, v in out.items()}


def operands(M, N, K, normal, device, batch=()):
    g = torch.Generator(device=device).manual_seed(M + 3 * N + 7 * K)
    if normal:
        return (torch.randn(batch + (M, K), generator=g, device=device), torch.randn(batch + (K, N), generator=g, device=device))
    return (torch.rand(batch + (M, K), generator=g, device=device) * 2 - 1, torch.rand(batch + (K, N), generator=g, device=device) * 2 - 1)


SHAPES = [(64, 64, 32), (63, 65, 33), (128, 127, 47), (257, 129, 64), (300, 520, 95), (70, 256, 100)]
LAYERS = [(1, 10, 34, 16, 64, 2, 3, 1), (2, 11, 19, 33, 70, 3, 1, 1), (1, 9, 9, 47, 129, 1, 1, 1), (1, 20, 41, 48, 40, 2, 1, 2),
          (2, 12, 37, 100, 130, 1, 1, 1)]


@pytest.mark.parametrize("normal", [False, True])
@pytest.mark.parametrize("shape", SHAPES)
def test_the_limit_tells_every_missing_product(shape, normal):
    a, b = operands(*shape, normal, "cpu")
    ref = a.double() @ b.double()
    sa, sb = slices(a), slices(b)
    parts = {p: sa[p[0]] @ sb[p[1]] for p in PRODUCTS}
    whole = sum(parts.values())
    assert rel(whole, ref) < 0.1 * limit(shape[2])
    for p in PRODUCTS:
        assert rel(whole - parts[p], ref) > limit(shape[2]), p


@pytest.mark.gpu
@pytest.mark.parametrize("shape", SHAPES)
@pytest.mark.parametrize("views", [None, (0, 0, 0), (1, 0, 0), (0, 1, 0), (1, 1, 1), (0, 0, 1)])
def test_products(shape, views):
    M, N, K = shape
    ta, tb, tc = views or (0, 0, 0)
    batch = 1 if views is None else 3
    inst, sizes = (mdh.MDH_MATMUL, shape) if views is None else (mdh.MDH_BMATMUL, (batch, M, N, K, ta, tb, tc))
    for normal in (False, True):
        a, b = operands(M, N, K, normal, "cuda", (batch,))
        refs = [a[i].double() @ b[i].double() for i in range(batch)]
        A, B = (a.transpose(1, 2).contiguous() if ta else a), (b.transpose(1, 2).contiguous() if tb else b)
        for p in split_candidates(inst, sizes, 2 if views is None else 3):
            C = torch.full((batch, N, M) if tc else (batch, M, N), float("nan"), device="cuda")
            if views is None:
                mdh.mdh_matmul(A[0], B[0], C[0], p, workspace(inst, sizes, p))
            else:
                mdh.mdh_matmul_ex(A, B, C, bool(ta), bool(tb), bool(tc), p, workspace(inst, sizes, p))
            for i in range(batch):
                assert rel(C[i].t() if tc else C[i], refs[i]) <= limit(K), (p.table(), i)


@pytest.mark.gpu
@pytest.mark.parametrize("case", LAYERS)
def test_convolutions(case):
    N, H, W, C, K, R, S, st = case
    P, Q = (H - R) // st + 1, (W - S) // st + 1
    g = torch.Generator(device="cuda").manual_seed(C * 11 + K)
    x = torch.randn((N, H, W, C), generator=g, device="cuda")
    f = torch.randn((K, R, S, C), generator=g, device="cuda")
    win = x.double().unfold(1, R, st).unfold(2, S, st).permute(0, 1, 2, 4, 5, 3).reshape(N * P * Q, R * S * C)
    ref = (win @ f.double().reshape(K, R * S * C).t().contiguous()).view(N, P, Q, K)
    sizes = (N, P, Q, K, C, R, S, st, st)
    cands = split_candidates(mdh.MDH_MCC, sizes, 4)
    assert cands
    for p in cands:
        out = torch.full((N, P, Q, K), float("nan"), device="cuda")
        mdh.mdh_mcc(x, f, out, (st, st), p, workspace(mdh.MDH_MCC, sizes, p))
        assert rel(out, ref) <= limit(R * S * C), p.table()


# a deep k in parts, with the workspace the default asks for and without: sums as accurate as one chain of them
@pytest.mark.gpu
@pytest.mark.parametrize("shape", [(90, 90, 8000), (40, 2000, 2000), (64, 64, 4096), (320, 900, 2500), (128, 300, 2001)])
def test_parts_of_a_deep_k(shape):
    a, b = operands(*shape, False, "cuda")
    for ws in (workspace(mdh.MDH_MATMUL, shape, None), None):
        C = torch.full((shape[0], shape[1]), float("nan"), device="cuda")
        mdh.mdh_matmul(a, b, C, None, ws)
        assert rel(C, a.double() @ b.double()) <= limit(shape[2])

"""Sums of one term through the kernels that carry an fp32 value as three bf16 values: a product with a permutation
(the identity, a delta filter, an image of one pixel) returns the other operand bit for bit, as fp32 arithmetic does,
and a product with a diagonal matrix is one multiplication.

The slices come back together without rounding if the smaller ones are added first: m + l = x - h is a float, and
h + (m + l) = x.  Bound of one multiplication: |m| <= 2^-8 |x|, |l| <= 2^-17 |x|, so the products left out (m l', l m',
l l') are at most (1 + 2^-10) 2^-24 |x x'|; the last addition cuts less than an ulp off (the bf16 matrix instruction
does not round to nearest), 2^-23 of the sum, the five before it, of sums below 2^-6 |x x'|, less than 2^-29 each.
"""
import pytest

import paper_2405_05118_amd as mdh

torch = pytest.importorskip("torch")

ONE_TERM = (3 + 2.0**-10 + 5 * 2.0**-5) * 2.0**-24


def is_split(inst, p):
    return p.prt[2][4] == 8 if inst == mdh.MDH_MCC else p.blk[p.D - 1] == 16


def tables(inst, sizes):
    """The default (None), which is one of the split kernels at these sizes, and every candidate of theirs."""
    cands = [mdh.mdh_candidate(inst, sizes, i) for i in range(mdh.mdh_num_candidates(inst, sizes))]
    assert is_split(inst, mdh.mdh_default_params(inst, sizes))
    return [None] + [p for p in cands if is_split(inst, p)]


def workspace(inst, sizes, p):
    n = mdh.mdh_workspace_size(inst, sizes, p)
    return torch.empty(n // 4, device="cuda") if n else None


def test_default_of_these_sizes():
    assert len(tables(mdh.MDH_BMATMUL, (2, 416, 416, 416, 0, 0, 0))) > 5
    assert len(tables(mdh.MDH_MATMUL, (832, 832, 832))) > 5
    assert len(tables(mdh.MDH_MCC, (2, 24, 40, 96, 96, 3, 3, 1, 1))) > 5


def values(shape, seed):
    """Every exponent from 2^-60 to 2^60, random mantissas."""
    g = torch.Generator(device="cuda").manual_seed(seed)
    m = torch.randint(-(1 << 24) + 1, 1 << 24, shape, generator=g, device="cuda").float()
    return torch.ldexp(m, torch.randint(-84, 37, shape, generator=g, device="cuda"))


@pytest.mark.gpu
@pytest.mark.parametrize("views", [None, (0, 0, 0), (1, 0, 0), (0, 1, 0), (1, 1, 0), (0, 0, 1), (1, 1, 1)])
def test_products_of_one_term(views):
    batch, n = (1, 832) if views is None else (2, 416)
    ta, tb, tc = views or (0, 0, 0)
    inst, sizes = (mdh.MDH_MATMUL, (n, n, n)) if views is None else (mdh.MDH_BMATMUL, (batch, n, n, n, ta, tb, tc))
    x, d = values((batch, n, n), 1), values((batch, n), 2)
    perm = torch.randperm(n, generator=torch.Generator().manual_seed(3)).cuda()
    P = torch.eye(n, device="cuda")[perm].expand(batch, n, n).contiguous()  # row i of P x is row perm[i] of x
    D = torch.diag_embed(d)
    for p in tables(inst, sizes):
        ws = workspace(inst, sizes, p)

        def product(a, b):
            a, b = (a.transpose(1, 2).contiguous() if ta else a), (b.transpose(1, 2).contiguous() if tb else b)
            c = torch.full((batch, n, n), float("nan"), device="cuda")
            if views is None:
                mdh.mdh_matmul(a[0], b[0], c[0], p, ws)
            else:
                mdh.mdh_matmul_ex(a, b, c, bool(ta), bool(tb), bool(tc), p, ws)
            return c.transpose(1, 2) if tc else c

        assert torch.equal(product(P, x), x[:, perm]), p and p.table()
        assert torch.equal(product(x, P)[:, :, perm], x), p and p.table()  # column perm[i] of x P is column i of x
        for got, ref in ((product(D, x), d[:, :, None].double() * x.double()), (product(x, D), x.double() * d[:, None, :].double())):
            assert float(((got.double() - ref).abs() / ref.abs().clamp(min=2.0**-100)).max()) <= ONE_TERM, p and p.table()


@pytest.mark.gpu
def test_convolutions_of_one_term():
    N, H, W, C, R = 2, 26, 42, 96, 3
    P, Q = H - R + 1, W - R + 1
    sizes = (N, P, Q, C, C, R, R, 1, 1)
    x, f = values((N, H, W, C), 4), values((C, R, R, C), 5)
    perm = torch.randperm(C, generator=torch.Generator().manual_seed(6)).cuda()
    delta = torch.zeros((C, R, R, C), device="cuda")
    delta[torch.arange(C), 1, 2, perm] = 1.0
    pixel = torch.zeros_like(x)
    pixel[1, 13, 17, 37] = 1.0
    want = torch.zeros((N, P, Q, C), device="cuda")
    for r in range(R):
        for s in range(R):
            want[1, 13 - r, 17 - s] = f[:, r, s, 37]
    for p in tables(mdh.MDH_MCC, sizes):
        ws = workspace(mdh.MDH_MCC, sizes, p)
        out = torch.full((N, P, Q, C), float("nan"), device="cuda")
        mdh.mdh_mcc(x, delta, out, (1, 1), p, ws)
        assert torch.equal(out, x[:, 1 : 1 + P, 2 : 2 + Q][..., perm]), p and p.table()
        out.fill_(float("nan"))
        mdh.mdh_mcc(pixel, f, out, (1, 1), p, ws)
        assert torch.equal(out, want), p and p.table()
        # one tap of one channel per output channel: a multiplication each
        for r, s in ((0, 0), (1, 2), (2, 1)):
            one = torch.zeros_like(f)
            one[torch.arange(C), r, s, perm] = f[torch.arange(C), r, s, perm]
            ref = x[:, r : r + P, s : s + Q][..., perm].double() * f[torch.arange(C), r, s, perm].double()
            out.fill_(float("nan"))
            mdh.mdh_mcc(x, one, out, (1, 1), p, ws)
            assert float(((out.double() - ref).abs() / ref.abs().clamp(min=2.0**-100)).max()) <= ONE_TERM, p and p.table()

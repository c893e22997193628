"""The kernels that carry an fp32 value as three bf16 values (six matrix products per multiply-add): tile edges,
reduction tails, views and split reductions against 64 bits, and the values such a sum does not carry.

Tolerance: the products left out are below (1 + 2^-10) 2^-24 of |a b| (test_split_exact), the six that are there are
exact, and every one of the fp32 accumulation steps (six per 16 terms, fewer than the K of a multiply-add chain, each
cutting less than an ulp off) adds at most 2^-23 of the running sum |a b|: (0.75 K + 1) 2^-24 of sum |a b|, below
K * 2^-24 from five terms on, as for the fp32 instructions.  That is an elementwise bound for edges, tails and parts;
test_split_accuracy has the limits that tell a missing product.
"""
import pytest

import paper_2405_05118_amd as mdh

torch = pytest.importorskip("torch")


def split_candidates(inst, sizes, kdim):
    all_ = [mdh.mdh_candidate(inst, sizes, i) for i in range(mdh.mdh_num_candidates(inst, sizes))]
    if inst == mdh.MDH_MCC:  # 16 input channels per matrix instruction, as eight register parts of two
        return [p for p in all_ if p.prt[2][kdim] == 8]
    return [p for p in all_ if p.blk[kdim] == 16]


def test_planner_of_the_split_kernels():
    sizes = (1000, 900, 777)
    cands = split_candidates(mdh.MDH_MATMUL, sizes, 2)
    assert len({(p.prt[4][0] * p.prt[2][0], p.prt[4][1] * p.prt[2][1]) for p in cands}) == 5
    p = cands[0]
    assert mdh.mdh_validate_params(mdh.MDH_MATMUL, sizes, p) == 0
    bad = p.copy()
    bad.blk[2] = 8
    assert mdh.mdh_validate_params(mdh.MDH_MATMUL, sizes, bad) != 0
    # fewer k than one k-tile, few channels: no split kernel
    assert not split_candidates(mdh.MDH_MATMUL, (300, 300, 31), 2)
    assert not split_candidates(mdh.MDH_MCC, (2, 20, 20, 64, 15, 3, 3, 1, 1), 4)
    assert split_candidates(mdh.MDH_MCC, (2, 20, 20, 64, 16, 3, 3, 1, 1), 4)


# the default splits a deep k further when the workspace it asks for is there, and does without when it is not
@pytest.mark.gpu
@pytest.mark.parametrize("shape", [(90, 90, 8000), (40, 2000, 2000), (64, 64, 4096), (320, 900, 2500), (128, 300, 2001)])
def test_matmul_default_with_and_without_workspace(shape):
    M, N, K = shape
    g = torch.Generator(device="cuda").manual_seed(K)
    A = torch.rand((M, K), generator=g, device="cuda") * 2 - 1
    B = torch.rand((K, N), generator=g, device="cuda") * 2 - 1
    ref = A.cpu().double() @ B.cpu().double()
    mag = A.cpu().double().abs() @ B.cpu().double().abs()
    n = mdh.mdh_workspace_size(mdh.MDH_MATMUL, shape)
    for ws in (None, torch.empty(max(n // 4 - 1, 1), device="cuda"), torch.empty(max(n // 4, 1), device="cuda")):
        C = torch.full((M, N), float("nan"), device="cuda")
        mdh.mdh_matmul(A, B, C, None, ws)
        assert float(((C.cpu().double() - ref).abs() / mag).max()) <= K * 2.0**-24


# M, N, K: one row less, exactly, and one more than tiles of 64 / 128 / 256; the shortest k, whole k-tiles, tails
@pytest.mark.gpu
@pytest.mark.parametrize("shape", [(64, 64, 32), (63, 65, 33), (128, 127, 47), (257, 129, 64), (300, 520, 95), (1, 256, 161)])
@pytest.mark.parametrize("views", [(0, 0, 0), (1, 0, 0), (0, 1, 0), (1, 1, 1), (0, 0, 1)])
def test_matmul_split_tiles(shape, views):
    M, N, K = shape
    ta, tb, tc = views
    batch = 3 if views != (0, 0, 0) else 1
    g = torch.Generator(device="cuda").manual_seed(M * 7 + K)
    A = torch.rand((batch, K, M) if ta else (batch, M, K), generator=g, device="cuda") * 2 - 1
    B = torch.rand((batch, N, K) if tb else (batch, K, N), generator=g, device="cuda") * 2 - 1
    a, b = (A.transpose(1, 2) if ta else A).cpu().double(), (B.transpose(1, 2) if tb else B).cpu().double()
    ref, mag = a @ b, a.abs() @ b.abs()
    plain = batch == 1
    inst, sizes = (mdh.MDH_MATMUL, shape) if plain else (mdh.MDH_BMATMUL, (batch, M, N, K, ta, tb, tc))
    cands = split_candidates(inst, sizes, 2 if plain else 3)
    assert cands
    for p in cands:
        C = torch.full((batch, N, M) if tc else (batch, M, N), float("nan"), device="cuda")
        n = mdh.mdh_workspace_size(inst, sizes, p)
        ws = torch.empty(n // 4, device="cuda") if n else None
        if plain:
            mdh.mdh_matmul(A[0], B[0], C[0], p, ws)
        else:
            mdh.mdh_matmul_ex(A, B, C, bool(ta), bool(tb), bool(tc), p, ws)
        got = (C.transpose(1, 2) if tc else C).cpu().double()
        assert float(((got - ref).abs() / mag).max()) <= K * 2.0**-24, p.table()


# N, H, W, C, K, R, S, stride: channel tails of both chunk sizes, edges of p, q and k, one tap, strides
@pytest.mark.gpu
@pytest.mark.parametrize("case", [(1, 10, 34, 16, 64, 3, 3, 1), (2, 11, 19, 33, 70, 3, 2, 1), (1, 9, 9, 47, 129, 1, 1, 1),
                                  (2, 17, 40, 70, 31, 5, 5, 2), (1, 14, 38, 64, 128, 7, 7, 1)])
def test_mcc_split_tiles(case):
    N, H, W, C, K, R, S, st = case
    P, Q = (H - R) // st + 1, (W - S) // st + 1
    g = torch.Generator(device="cuda").manual_seed(C * 11 + K)
    x = torch.randn((N, H, W, C), generator=g, device="cuda")
    f = torch.randn((K, R, S, C), generator=g, device="cuda")
    win = x.cpu().double().unfold(1, R, st).unfold(2, S, st).permute(0, 1, 2, 4, 5, 3).reshape(N * P * Q, R * S * C)
    flat = f.cpu().double().reshape(K, R * S * C).t()
    ref, mag = (win @ flat).view(N, P, Q, K), (win.abs() @ flat.abs()).view(N, P, Q, K)
    sizes = (N, P, Q, K, C, R, S, st, st)
    cands = split_candidates(mdh.MDH_MCC, sizes, 4)
    assert cands
    for p in cands:
        out = torch.full((N, P, Q, K), float("nan"), device="cuda")
        n = mdh.mdh_workspace_size(mdh.MDH_MCC, sizes, p)
        mdh.mdh_mcc(x, f, out, (st, st), p, torch.empty(n // 4, device="cuda") if n else None)
        err = float(((out.cpu().double() - ref).abs() / mag).max())
        assert err <= R * S * C * 2.0**-24, (p.table(), err)


# Values a sum of three bf16 values does not carry: the outputs they enter are those of the fp32 instructions.
@pytest.mark.gpu
@pytest.mark.parametrize("what", ["inf", "nan", "largest", "tiny rows", "tiny against huge", "subnormal", "zero rows"])
def test_values_beyond_the_split(what):
    M, N, K = 200, 150, 160
    g = torch.Generator(device="cuda").manual_seed(3)
    A = torch.rand((M, K), generator=g, device="cuda") * 2 - 1
    B = torch.rand((K, N), generator=g, device="cuda") * 2 - 1
    if what == "inf":
        A[3, 5], A[3, 6], B[7, 9], A[70, 1] = float("inf"), float("inf"), float("-inf"), float("-inf")
        B[5, 4] = 0.0  # inf * 0
    elif what == "nan":
        A[130, 0], B[159, 149] = float("nan"), float("nan")
    elif what == "largest":
        A[11] = torch.finfo(torch.float32).max
        B[:, 5] = B[:, 5] * 1e-3
    elif what == "tiny rows":
        A[20:40] *= 1e-36
    elif what == "tiny against huge":
        A[20:40] *= 1e-36
        B *= 1e30
    elif what == "subnormal":
        A[20:40] *= 1e-40
        B *= 1e25
    else:
        A[64:128] = 0.0
    fp32 = next(q for q in (mdh.mdh_candidate(mdh.MDH_MATMUL, (M, N, K), i) for i in range(mdh.mdh_num_candidates(mdh.MDH_MATMUL, (M, N, K))))
                if q.blk[2] == 2 and q.prt[4][2] == 1 and q.prt[3][2] == 1)
    want = torch.empty((M, N), device="cuda")
    mdh.mdh_matmul(A, B, want, fp32)
    mag = A.cpu().double().abs() @ B.cpu().double().abs()
    finite = torch.isfinite(want.cpu())
    x, f = A.view(1, 1, M, K), B.t().contiguous().view(N, 1, 1, K)
    results = []
    for p in split_candidates(mdh.MDH_MATMUL, (M, N, K), 2):
        if p.prt[3][2] == 1:
            C = torch.full((M, N), 7.0, device="cuda")
            mdh.mdh_matmul(A, B, C, p)
            results.append((C, p))
    for p in split_candidates(mdh.MDH_MCC, (1, 1, M, N, K, 1, 1, 1, 1), 4):  # the same product as a 1 x 1 layer
        if p.prt[3][4] == 1:
            C = torch.full((1, 1, M, N), 7.0, device="cuda")
            mdh.mdh_mcc(x, f, C, (1, 1), p)
            results.append((C.view(M, N), p))
    assert len(results) > 5
    for C, p in results:
        got = C.cpu()
        assert torch.equal(torch.isnan(got), torch.isnan(want.cpu())), p.table()
        assert torch.equal(got[torch.isinf(got)], want.cpu()[torch.isinf(want.cpu())]), p.table()
        ref = (A.cpu().double() @ B.cpu().double())[finite]
        err = (got[finite].double() - ref).abs()
        # an output has the accuracy of fp32, or is off by what fp32 cannot hold (subnormal results)
        assert bool((err <= K * 2.0**-24 * mag[finite] + K * 2.0**-149).all()), p.table()

"""Tables of the kernels that carry a value as three bf16 values: what the planner refuses and what it offers."""
import os
import subprocess
import sys

import pytest

import paper_2405_05118_amd as mdh

MAX_D = 10
ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

# every entry of the table that the k-tile or the part of k is computed from, at values whose products wrap to nothing,
# to a valid tile or to a negative one; one table a line, so that a crash names its table
HUGE = """
import paper_2405_05118_amd as mdh
for inst, sizes, k in ((mdh.MDH_MATMUL, (256, 256, 256), 2), (mdh.MDH_BMATMUL, (2, 256, 256, 256, 0, 1, 0), 3),
                       (mdh.MDH_BMATMUL, (2, 256, 256, 256, 0, 1, 1), 3), (mdh.MDH_MCC, (1, 16, 32, 64, 64, 3, 3, 1, 1), 4)):
    cands = [mdh.mdh_candidate(inst, sizes, i) for i in range(mdh.mdh_num_candidates(inst, sizes))]
    p = next(p for p in cands if (p.prt[2][4] == 8 if inst == mdh.MDH_MCC else p.blk[k] == 16))
    for layer in range(6):
        for d in range(p.D):
            for v in (1 << 25, 1 << 26, (1 << 26) + 1, 1 << 27, (1 << 27) + 1, 1 << 28, (1 << 28) + 1, (1 << 28) + 2, 1 << 30, (1 << 31) - 1):
                q = p.copy()
                q.ragged = 1
                q.prt[layer][d] = v
                print(inst, sizes, layer, d, v, flush=True)
                assert mdh.mdh_validate_params(inst, sizes, q) != 0
print("all refused")
"""


def test_tables_whose_products_wrap_are_refused():
    r = subprocess.run([sys.executable, "-c", HUGE], cwd=ROOT, capture_output=True, text=True, timeout=300)
    assert r.returncode == 0 and r.stdout.endswith("all refused\n"), (r.returncode, r.stdout[-200:], r.stderr[-500:])


# the tables of the few-channel kernels, with fp32 instructions and with slices
FEW = """
import paper_2405_05118_amd as mdh
sizes = (2, 40, 43, 64, 3, 7, 7, 1, 1)
cands = [mdh.mdh_candidate(mdh.MDH_MCC, sizes, i) for i in range(mdh.mdh_num_candidates(mdh.MDH_MCC, sizes))]
for region in (0, 1):
    p = next(p for p in cands if p.blk[4] == 1 and p.in_region[0] == region)
    for layer in range(6):
        for d in range(p.D):
            for v in [1 << b for b in range(12, 31)] + [(1 << b) + 1 for b in range(25, 31)] + [(1 << 31) - 1]:
                q = p.copy()
                q.ragged = 1
                q.prt[layer][d] = v
                print(region, layer, d, v, flush=True)
                assert mdh.mdh_validate_params(mdh.MDH_MCC, sizes, q) != 0
print("all refused")
"""


def test_few_channel_tables_whose_products_wrap_are_refused():
    r = subprocess.run([sys.executable, "-c", FEW], cwd=ROOT, capture_output=True, text=True, timeout=300)
    assert r.returncode == 0 and r.stdout.endswith("all refused\n"), (r.returncode, r.stdout[-200:], r.stderr[-500:])


# the few-channel kernel on slices is for images of less than 2^28 values: the largest that the sizes allow counts, also where
# one output a row or column leaves the stride open, up to products beyond 64 bits
@pytest.mark.parametrize("P, Q, C, stride, offered", [(112, 112, 3, 2, True), (1, 1, 3, 9000, True), (1, 1, 3, 10000, False),
                                                      (9000, 9000, 4, 1, False), (1, 1, 1, 2**31 - 1, False), (1, 1, 3, 2**31 - 1, False),
                                                      (2, 2, 1, 2**31 - 1, False), (1, 1, 2, 2**30 + 2**29, False)])
def test_few_channel_images_beyond_32_bits(P, Q, C, stride, offered):
    sizes = (1, P, Q, 64, C, 7, 7, stride, stride)
    tables = [mdh.mdh_candidate(mdh.MDH_MCC, sizes, i) for i in range(mdh.mdh_num_candidates(mdh.MDH_MCC, sizes))]
    assert any(p.blk[4] == 1 and p.in_region[0] == 0 for p in tables) == offered


# What a call without a table runs: the default's table, but for few channels the kernel on slices where its matrix
# instructions take at most two thirds of the time (nine tenths below 2^24 outputs) and a sum has 18 terms or more.
@pytest.mark.parametrize("sizes, sliced", [
    ((16, 112, 112, 64, 3, 7, 7, 2, 2), True), ((1, 112, 112, 64, 3, 7, 7, 2, 2), True), ((16, 224, 224, 64, 3, 5, 5, 1, 1), True),
    ((16, 222, 222, 64, 4, 3, 3, 1, 1), True), ((16, 222, 222, 64, 3, 3, 3, 1, 1), False), ((8, 222, 222, 32, 3, 3, 3, 1, 1), True),
    ((16, 220, 220, 64, 2, 5, 5, 1, 1), False), ((4, 60, 60, 32, 2, 5, 5, 1, 1), True), ((4, 60, 60, 32, 2, 3, 3, 1, 1), True), ((16, 222, 222, 64, 2, 3, 3, 1, 1), False),
    ((4, 60, 60, 32, 1, 3, 3, 1, 1), False), ((4, 60, 60, 32, 2, 1, 7, 1, 1), False),
])
def test_what_a_call_without_a_table_runs(sizes, sliced):
    p, d = mdh.mdh_call_params(mdh.MDH_MCC, sizes), mdh.mdh_default_params(mdh.MDH_MCC, sizes)
    assert p.blk[4] == d.blk[4] == 1 and d.in_region[0] == 1 and (p.in_region[0] == 0) == sliced
    assert sliced or bytes(p) == bytes(d)
    assert mdh.mdh_validate_params(mdh.MDH_MCC, sizes, p) == 0 and mdh.mdh_workspace_size(mdh.MDH_MCC, sizes) == 0


@pytest.mark.parametrize("inst, sizes", [
    (mdh.MDH_MATMUL, (300, 200, 100)), (mdh.MDH_MATMUL, (4096, 4096, 4096)), (mdh.MDH_MATMUL, (3, 500, 4000)),
    (mdh.MDH_MCC, (16, 56, 56, 64, 64, 3, 3, 1, 1)), (mdh.MDH_STENCIL, (30, 40, 50)), (mdh.MDH_CUSTOM_REDUCE, (5000, 9000, 8)),
    (mdh.MDH_BMATMUL, (4, 60, 70, 80, 0, 1, 0)), (mdh.MDH_DOT, (1 << 20,)), (mdh.MDH_MATVEC, (100, 200)), (mdh.MDH_SCAN, (4, 10000)),
    (mdh.MDH_MCC_CAPSULE, (1, 8, 8, 16, 4, 3, 3, 1, 1))])
def test_elsewhere_that_is_the_default(inst, sizes):
    assert bytes(mdh.mdh_call_params(inst, sizes)) == bytes(mdh.mdh_default_params(inst, sizes))


# the default's tile in column bands, and what the small-M kernel stands in front of, where the split kernels or parts
# of k have become the default: WG, WAVE and VGPR parts of (i, j, k), and the loop order's first entry
@pytest.mark.parametrize("sizes, wg, wave, vgpr, first", [
    ((496, 139, 20778), (8, 3, 16), (2, 2, 1), (1, 1, 1), 3 * MAX_D + 1),
    ((87, 5853, 17022), (2, 92, 2), (2, 2, 1), (1, 1, 1), 3 * MAX_D + 1),
    ((1, 1861, 5605), (1, 117, 2), (1, 1, 8), (1, 1, 4), 3 * MAX_D),
])
def test_candidates_beside_the_default(sizes, wg, wave, vgpr, first):
    assert any((tuple(p.prt[3][:3]), tuple(p.prt[4][:3]), tuple(p.prt[2][:3])) == (wg, wave, vgpr) and p.order[0] == first and p.blk[2] != 16
               for p in (mdh.mdh_candidate(mdh.MDH_MATMUL, sizes, i) for i in range(mdh.mdh_num_candidates(mdh.MDH_MATMUL, sizes))))


# the default of these sizes asks for a workspace it can do without, also where the caller passes its table
@pytest.mark.gpu
@pytest.mark.parametrize("shape", [(90, 90, 8000), (40, 2000, 2000), (128, 300, 5001)])
def test_table_of_the_default_without_workspace(shape):
    import torch

    M, N, K = shape
    p = mdh.mdh_default_params(mdh.MDH_MATMUL, shape)
    assert mdh.mdh_workspace_size(mdh.MDH_MATMUL, shape, p) > 0
    A, B = torch.ones((M, K), device="cuda"), torch.ones((K, N), device="cuda")
    for q in (None, p):
        C = torch.full((M, N), float("nan"), device="cuda")
        mdh.mdh_matmul(A, B, C, q, None)
        assert bool((C == K).all())
    # another table that splits k is taken as it stands
    cands = [mdh.mdh_candidate(mdh.MDH_MATMUL, shape, i) for i in range(1, mdh.mdh_num_candidates(mdh.MDH_MATMUL, shape))]
    with pytest.raises(mdh.MdhError) as e:
        mdh.mdh_matmul(A, B, C, next(q for q in cands if q.prt[3][2] == 2), None)
    assert e.value.status == 5


# Products and layers whose default asks for a workspace and did not always: a call without a table runs with fewer parts where
# it is missing or holds only some, and is close to 64 bits all the same (as in test_split_k).
LESS = [(mdh.MDH_MATMUL, (15890, 62, 1233)), (mdh.MDH_MATMUL, (12627, 59, 976)), (mdh.MDH_MCC, (9, 28, 28, 248, 464, 7, 7, 1, 1)),
        (mdh.MDH_MCC, (3, 13, 16, 487, 47, 3, 3, 2, 2)), (mdh.MDH_MCC, (4, 20, 20, 77, 174, 1, 1, 1, 1)), (mdh.MDH_MCC, (8, 10, 15, 332, 405, 3, 3, 1, 1)),
        (mdh.MDH_BMATMUL, (1, 12677, 62, 1283, 1, 0, 0)), (mdh.MDH_BMATMUL, (5, 2934, 52, 1067, 0, 1, 1))]


@pytest.mark.gpu
@pytest.mark.parametrize("inst,sizes", LESS)
@pytest.mark.parametrize("parts", [0, 1, 2, 3])
def test_default_with_less_workspace(inst, sizes, parts):
    import torch

    g = torch.Generator(device="cuda").manual_seed(parts + sizes[0])
    rand = lambda *shape: torch.rand(shape, generator=g, device="cuda") * 2 - 1
    if inst == mdh.MDH_MCC:
        n, P, Q, K, C, R, S, st, _ = sizes
        a, b = rand(n, (P - 1) * st + R, (Q - 1) * st + S, C), rand(K, R, S, C)
        ref, mag, terms = torch.zeros((n * P * Q, K), dtype=torch.float64, device="cuda"), 0.0, C * R * S
        for r in range(R):
            for s in range(S):
                tap = a[:, r : r + (P - 1) * st + 1 : st, s : s + (Q - 1) * st + 1 : st].reshape(-1, C).double()
                w = b[:, r, s].double().t().contiguous()
                ref += tap @ w
                mag = mag + tap.abs() @ w.abs()
        ref, mag = ref.view(n, P, Q, K), mag.view(n, P, Q, K)
        call = lambda out, p, ws: mdh.mdh_mcc(a, b, out, (st, st), p, ws)
    else:
        batch, M, N, terms, ta, tb, tc = sizes if inst == mdh.MDH_BMATMUL else (1, *sizes, 0, 0, 0)
        a, b = rand(batch, M, terms), rand(batch, terms, N)
        ref = torch.stack([a[i].double() @ b[i].double() for i in range(batch)])
        mag = torch.stack([a[i].double().abs() @ b[i].double().abs() for i in range(batch)])
        ref, mag = (ref.transpose(1, 2), mag.transpose(1, 2)) if tc else (ref, mag)
        A, B = (a.transpose(1, 2).contiguous() if ta else a), (b.transpose(1, 2).contiguous() if tb else b)
        if inst == mdh.MDH_BMATMUL:
            call = lambda out, p, ws: mdh.mdh_matmul_ex(A, B, out, bool(ta), bool(tb), bool(tc), p, ws)
        else:
            call = lambda out, p, ws: mdh.mdh_matmul(A[0], B[0], out[0], p, ws)
    need, n = mdh.mdh_workspace_size(inst, sizes), ref.numel()
    assert need > 0 and need % (n * 4) == 0
    table = mdh.mdh_default_params(inst, sizes)
    for p in (None, table):
        out = torch.full(ref.shape, float("nan"), device="cuda")
        room = torch.full((parts * n + 64,), 7.0, device="cuda")  # 64 guard words
        if p and inst != mdh.MDH_MATMUL and parts * n * 4 < need:  # a table is taken as it stands, but MatMul's default
            with pytest.raises(mdh.MdhError) as e:
                call(out, p, room[: parts * n] if parts else None)
            assert e.value.status == 5
            continue
        call(out, p, room[: parts * n] if parts else None)
        assert bool(((out.double() - ref).abs() <= terms * 2.0**-24 * mag).all())
        assert bool((room[parts * n :] == 7.0).all())


# a part of c is a chain in one accumulator, and a longer one is further from 64 bits: the number of parts that the estimate
# of the tiles alone would take is half of these or less
@pytest.mark.parametrize("sizes,parts", [
    ((5, 19, 24, 235, 121, 3, 3, 1, 1), 4), ((3, 55, 56, 51, 180, 5, 5, 1, 1), 4), ((9, 10, 15, 489, 127, 3, 3, 1, 1), 4), ((5, 8, 9, 229, 339, 3, 3, 1, 1), 8),
    ((2, 19, 20, 497, 67, 7, 7, 1, 1), 2), ((14, 7, 12, 57, 279, 1, 1, 1, 1), 4), ((7, 26, 26, 397, 110, 5, 5, 2, 2), 2)])
def test_parts_of_c_stay_short(sizes, parts):
    p = mdh.mdh_default_params(mdh.MDH_MCC, sizes)
    assert p.prt[2][4] == 8 and p.prt[3][4] >= parts


@pytest.mark.parametrize("sizes,parts", [((25978, 49, 1755), 2), ((14058, 51, 1529), 4), ((19632, 55, 887), 2), ((54, 21694, 783), 2), ((1844, 53, 10969), 32)])
def test_parts_of_k_stay_short(sizes, parts):
    for inst, s, k in ((mdh.MDH_MATMUL, sizes, 2), (mdh.MDH_BMATMUL, (1, *sizes, 0, 0, 0), 3)):
        p = mdh.mdh_default_params(inst, s)
        assert p.blk[k] == 16 and p.prt[3][k] * p.prt[4][k] >= parts, inst


# the tiles in chunks of 32 channels cut c as evenly as those in chunks of 16, so that their chains are as short
@pytest.mark.gpu
@pytest.mark.parametrize("sizes,parts", [((2, 20, 24, 64, 66, 5, 5, 1, 1), 2), ((1, 9, 33, 70, 134, 3, 3, 2, 2), 2), ((1, 18, 18, 32, 129, 3, 3, 1, 1), 2),
                                         ((1, 18, 18, 32, 226, 3, 3, 1, 1), 4)])
def test_parts_of_c_are_even(sizes, parts):
    import torch

    n, P, Q, K, C, R, S, st, _ = sizes
    g = torch.Generator(device="cuda").manual_seed(C)
    x = torch.randn((n, (P - 1) * st + R, (Q - 1) * st + S, C), generator=g, device="cuda")
    f = torch.randn((K, R, S, C), generator=g, device="cuda")
    ref = torch.zeros((n * P * Q, K), dtype=torch.float64, device="cuda")
    for r in range(R):
        for s in range(S):
            ref += x[:, r : r + (P - 1) * st + 1 : st, s : s + (Q - 1) * st + 1 : st].reshape(-1, C).double() @ f[:, r, s].double().t().contiguous()
    error = {16: [], 32: []}
    for p in (mdh.mdh_candidate(mdh.MDH_MCC, sizes, i) for i in range(mdh.mdh_num_candidates(mdh.MDH_MCC, sizes))):
        if p.blk[4] == 2 and p.prt[2][4] == 8 and p.prt[3][4] == parts:
            out = torch.full((n, P, Q, K), float("nan"), device="cuda")
            mdh.mdh_mcc(x, f, out, (st, st), p, torch.empty(parts * out.numel(), device="cuda"))
            error[16 * p.prt[1][4]].append(float((out.view(-1, K).double() - ref).norm()))
    assert error[16] and error[32]
    assert max(error[32]) <= 1.03 * min(error[16])  # every tile takes the same parts, and the same steps of 16 in them

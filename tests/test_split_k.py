"""MatMul on three-slice values with k over the wavefronts of a workgroup: tiles that are moved inside at the edges, parts of
k that are no whole number of steps, every view, and values that the split does not carry, against 64 bits.

Tolerance: of a sum of K products at most K 2^-24 of the magnitudes' sum, as for every kernel on slices; few terms as
derived in test_split_exact (3 x 2^-24 a product, and the roundings that bring the parts of k together, one a wavefront).
"""
import pytest

import paper_2405_05118_amd as mdh
from test_split_exact import workspace
from test_split_special import WHAT, check, plant, sums

torch = pytest.importorskip("torch")


TILES = ((2, 2, 8), (2, 2, 4), (2, 3, 4), (3, 2, 4), (3, 3, 4), (1, 2, 8), (2, 1, 8), (1, 1, 8))  # blocks, wavefronts


def table(inst, sizes, tile, S):
    """A table with k over the wavefronts, made from one that the planner offers."""
    k = 2 if inst == mdh.MDH_MATMUL else 3
    q = next(p for p in (mdh.mdh_candidate(inst, sizes, i) for i in range(mdh.mdh_num_candidates(inst, sizes))) if p.blk[k] == 16 and p.order[0] % 10 == 0)
    p = q.copy()
    mi, ni, w = tile if k == 2 or not sizes[6] else (tile[1], tile[0], tile[2])  # C transposed: the other order
    for layer in range(6):
        for d in range(k + 1):
            p.prt[layer][d] = 1
    if k == 3:
        p.prt[3][0] = sizes[0]
    M, N, K = sizes[k - 2 : k + 1]
    p.prt[3][k - 2], p.prt[3][k - 1], p.prt[3][k] = -(-M // (32 * mi)), -(-N // (32 * ni)), S
    p.prt[4][k], p.prt[0][k] = w, -(-(-(-K // (S * w))) // 32)
    p.prt[2][k - 2], p.prt[2][k - 1], p.prt[2][k] = mi, ni, 2
    p.in_region[0] = p.in_region[1] = 2
    p.out_region, p.ragged = 1, 1
    return p


def tables(inst, sizes):
    """Every tile that lies inside the output, in one, two and four parts of k where the last has two steps."""
    all_ = [table(inst, sizes, t, S) for t in TILES for S in (1, 2, 4)]
    return [p for p in all_ if mdh.mdh_validate_params(inst, sizes, p) == 0]


def tile(p):
    k = p.D - 1
    return p.prt[2][k - 2], p.prt[2][k - 1], p.prt[4][k]


def test_planner_accepts_and_refuses():
    assert {tile(p) for p in tables(mdh.MDH_MATMUL, (300, 300, 300))} == set(TILES)
    assert {p.prt[3][2] for p in tables(mdh.MDH_MATMUL, (300, 300, 320))} == {1, 2, 4}
    # a tile has to lie inside the output, a part of k holds two steps
    assert {tile(p)[:2] for p in tables(mdh.MDH_BMATMUL, (2, 95, 64, 300, 0, 1, 0))} == {(2, 2), (1, 2), (2, 1), (1, 1)}
    assert {tile(p)[:2] for p in tables(mdh.MDH_BMATMUL, (2, 95, 64, 300, 0, 1, 1))} == {(2, 2), (1, 2), (2, 1), (1, 1)}
    assert {p.prt[3][2] for p in tables(mdh.MDH_MATMUL, (300, 300, 47))} == {1}
    assert not tables(mdh.MDH_MATMUL, (31, 300, 300))
    for inst, sizes, k in ((mdh.MDH_MATMUL, (256, 256, 256), 2), (mdh.MDH_BMATMUL, (2, 256, 256, 256, 0, 1, 1), 3)):
        p = tables(inst, sizes)[0]
        for layer, d, v in ((4, k, 3), (4, k, 16), (4, k - 1, 2), (1, k, 2), (2, k, 4), (3, k, 9), (2, k - 1, (1 << 27) + 2), (4, k, (1 << 30) + 4)):
            q = p.copy()
            q.prt[layer][d] = v
            assert mdh.mdh_validate_params(inst, sizes, q) != 0, (layer, d, v)
        for blk in (2, 8, 32):
            q = p.copy()
            q.blk[k] = blk
            assert mdh.mdh_validate_params(inst, sizes, q) != 0, blk
    # the default of outputs of about a tile a compute unit, and candidates that are worth trying
    for inst, sizes in ((mdh.MDH_MATMUL, (1021, 1531, 777)), (mdh.MDH_BMATMUL, (8, 200, 333, 650, 0, 1, 0))):
        assert tile(mdh.mdh_default_params(inst, sizes))[2] > 1
        cands = [mdh.mdh_candidate(inst, sizes, i) for i in range(mdh.mdh_num_candidates(inst, sizes))]
        assert len({tile(p) for p in cands if p.blk[p.D - 1] == 16 and tile(p)[2] > 1}) > 1


# one tile, one row or column more, tiles that overlap by all but one row; two steps of 16, tails of either half of a chunk,
# fewer steps than wavefronts, parts of k
@pytest.mark.gpu
@pytest.mark.parametrize("shape", [(32, 32, 32), (64, 65, 33), (97, 96, 47), (127, 161, 129), (70, 100, 272), (193, 33, 535), (129, 191, 800)])
@pytest.mark.parametrize("views", [None, (0, 0, 0), (1, 0, 0), (0, 1, 0), (1, 1, 0), (0, 0, 1), (1, 1, 1)])
def test_tiles_views_and_parts(shape, views):
    M, N, K = shape
    ta, tb, tc = views or (0, 0, 0)
    batch = 1 if views is None else 3
    inst, sizes = (mdh.MDH_MATMUL, shape) if views is None else (mdh.MDH_BMATMUL, (batch, M, N, K, ta, tb, tc))
    g = torch.Generator(device="cuda").manual_seed(M * 7 + K)
    a = torch.rand((batch, M, K), generator=g, device="cuda") * 2 - 1
    b = torch.rand((batch, K, N), generator=g, device="cuda") * 2 - 1
    A, B = (a.transpose(1, 2).contiguous() if ta else a), (b.transpose(1, 2).contiguous() if tb else b)
    cands = tables(inst, sizes)
    assert cands and (K < 256 or len({p.prt[3][p.D - 1] for p in cands}) > 1)
    for p in cands:
        C = torch.full((batch, N, M) if tc else (batch, M, N), float("nan"), device="cuda")
        guard = torch.cat([C.flatten(), torch.full((256,), 7.0, device="cuda")])  # nothing beyond the output is written
        C = guard[: C.numel()].view(C.shape)
        if views is None:
            mdh.mdh_matmul(A[0], B[0], C[0], p, workspace(inst, sizes, p))
        else:
            mdh.mdh_matmul_ex(A, B, C, bool(ta), bool(tb), bool(tc), p, workspace(inst, sizes, p))
        for i in range(batch):
            ref, mag = sums(a[i], b[i])
            got = (C[i].t() if tc else C[i]).double()
            assert bool(((got - ref).abs() <= K * 2.0**-24 * mag).all()), (p.table(), i)
        assert bool((guard[C.numel() :] == 7.0).all())


@pytest.mark.gpu
@pytest.mark.parametrize("what", WHAT + ["zero rows"])
@pytest.mark.parametrize("views", [(0, 0, 0), (1, 0, 0), (0, 1, 0), (1, 1, 1)])
def test_special_values(what, views):
    M, N, K = 150, 130, 535  # tiles overlap in both directions
    ta, tb, tc = views
    inst, sizes = mdh.MDH_BMATMUL, (2, M, N, K, ta, tb, tc)
    g = torch.Generator(device="cuda").manual_seed(len(what))
    a = torch.rand((2, M, K), generator=g, device="cuda") * 2 - 1
    b = torch.rand((2, K, N), generator=g, device="cuda") * 2 - 1
    if what == "zero rows":
        a[1, 20:90], b[1, :, 100:] = 0.0, 0.0
    else:
        plant(a[1], b[1], what, K)
    refs = [sums(a[i], b[i]) for i in range(2)]
    A, B = (a.transpose(1, 2).contiguous() if ta else a), (b.transpose(1, 2).contiguous() if tb else b)
    for p in tables(inst, sizes):
        C = torch.full((2, N, M) if tc else (2, M, N), 7.0, device="cuda")
        mdh.mdh_matmul_ex(A, B, C, bool(ta), bool(tb), bool(tc), p, workspace(inst, sizes, p))
        for i in range(2):
            check(C[i].t() if tc else C[i], *refs[i], K, (p.table(), i))


@pytest.mark.gpu
def test_a_permutation_is_exact_and_single_terms_round_once():
    n = 200
    sizes = (n, n, n)
    g = torch.Generator(device="cuda").manual_seed(1)
    x = (torch.rand((n, n), generator=g, device="cuda") * 2 - 1) * torch.exp2(torch.randint(-60, 60, (n, n), generator=g, device="cuda").float())
    perm = torch.eye(n, device="cuda")[torch.randperm(n, generator=g, device="cuda")]
    scale = torch.rand((n, 1), generator=g, device="cuda") + 0.5
    for p in tables(mdh.MDH_MATMUL, sizes):
        out = torch.full((n, n), 7.0, device="cuda")
        mdh.mdh_matmul(perm, x, out, p, workspace(mdh.MDH_MATMUL, sizes, p))
        assert torch.equal(out, perm @ x), p.table()
        mdh.mdh_matmul(perm * scale, x, out, p, workspace(mdh.MDH_MATMUL, sizes, p))
        ref, mag = sums(perm * scale, x)
        assert bool(((out.double() - ref).abs() <= (ONE_TERM if apart(p) else 3.0) * 2.0**-24 * mag).all()), p.table()


# Tiles of one or two blocks sum h h', which 16 bits hold exactly, apart: the seven smaller products, below 2^-7 of it
# together, are cut off at 2^-30 each, the sum of both is rounded once, and l l' (2^-34) is left out.
ONE_TERM = 1 + 7 * 2.0**-6 + 2.0**-10


def apart(p):
    return tile(p)[0] * tile(p)[1] <= 2


# Sums of few terms, as close to 64 bits as on the fp32 instructions with k over as many wavefronts.  Limit: over 12 times 65536
# outputs the ratio of the two errors was 1.000 for one term, 0.88 to 0.99 for 2 to 32 and less beyond; six products are at 1.026
# for one term, and one accumulator for all of them (MCC of few channels) at 1.4 for one and 1.8 for eight.
@pytest.mark.gpu
@pytest.mark.parametrize("terms", [1, 2, 3, 8, 32, 512])
def test_sums_of_few_terms(terms):
    sizes = M, N, K = 256, 256, 512
    g = torch.Generator(device="cuda").manual_seed(terms)
    at = torch.stack([torch.randperm(K, generator=g, device="cuda")[:terms] for _ in range(M)])
    a = torch.zeros((M, K), device="cuda").scatter_(1, at, torch.randn((M, terms), generator=g, device="cuda"))
    b = torch.randn((K, N), generator=g, device="cuda")
    ref = a.double() @ b.double()

    def error(p):
        out = torch.full((M, N), float("nan"), device="cuda")
        mdh.mdh_matmul(a, b, out, p, workspace(mdh.MDH_MATMUL, sizes, p))
        return float((out.double() - ref).norm())

    cands = [mdh.mdh_candidate(mdh.MDH_MATMUL, sizes, i) for i in range(mdh.mdh_num_candidates(mdh.MDH_MATMUL, sizes))]
    fp32 = next(p for p in cands if p.blk[2] != 16 and p.prt[4][2] == 8 and p.prt[3][2] == 1)
    tiles = [p for p in tables(mdh.MDH_MATMUL, sizes) if apart(p) and p.prt[3][2] == 1]
    assert len(tiles) == 3
    for p in tiles:
        assert error(p) <= 1.01 * error(fp32), p.table()


# Small batches and outputs of few tiles whose default is these tiles (K from 64 on), and the line: close to 64 bits through the
# default, and tables with fp32 instructions to choose instead.
SMALL = [(2, 64, 64, 64, 0, 0, 0), (1, 33, 33, 64, 0, 0, 0), (3, 70, 90, 65, 0, 1, 0), (5, 97, 61, 100, 1, 0, 1), (4, 203, 171, 127, 1, 1, 0), (4, 203, 171, 183, 0, 1, 0)]


@pytest.mark.parametrize("sizes", SMALL)
def test_default_of_small_batches(sizes):
    p = mdh.mdh_default_params(mdh.MDH_BMATMUL, sizes)
    assert p.blk[3] == 16 and apart(p) and tile(p)[2] == 8 and mdh.mdh_workspace_size(mdh.MDH_BMATMUL, sizes) == 0
    cands = [mdh.mdh_candidate(mdh.MDH_BMATMUL, sizes, i) for i in range(mdh.mdh_num_candidates(mdh.MDH_BMATMUL, sizes))]
    assert any(p.blk[3] == 2 for p in cands)


def test_line_of_small_batches():
    for sizes, split in (((2, 64, 64, 63, 0, 0, 0), False), ((2, 64, 64, 64, 0, 0, 0), True), ((2, 31, 64, 64, 0, 0, 0), False),
                         ((64, 512, 512, 100, 0, 0, 0), False)):
        assert (mdh.mdh_default_params(mdh.MDH_BMATMUL, sizes).blk[3] == 16) == split, sizes
    p = mdh.mdh_default_params(mdh.MDH_MATMUL, (288, 320, 2880))
    assert p.blk[2] == 16 and apart(p)
    assert mdh.mdh_default_params(mdh.MDH_MATMUL, (512, 512, 512)).blk[2] == 2


@pytest.mark.gpu
@pytest.mark.parametrize("sizes", SMALL)
def test_small_batches_are_close(sizes):
    batch, M, N, K, ta, tb, tc = sizes
    g = torch.Generator(device="cuda").manual_seed(K)
    a = torch.rand((batch, M, K), generator=g, device="cuda") * 2 - 1
    b = torch.rand((batch, K, N), generator=g, device="cuda") * 2 - 1
    A, B = (a.transpose(1, 2).contiguous() if ta else a), (b.transpose(1, 2).contiguous() if tb else b)
    C = torch.full((batch, N, M) if tc else (batch, M, N), float("nan"), device="cuda")
    mdh.mdh_matmul_ex(A, B, C, bool(ta), bool(tb), bool(tc))
    # 1.8e-8 sqrt(K) is what fp32 sums of random products show, 1.2e-7 at the least
    for i in range(batch):
        ref = a[i].double() @ b[i].double()
        assert float(((C[i].t() if tc else C[i]).double() - ref).norm() / ref.norm()) <= max(1.2e-7, 1.8e-8 * K**0.5)

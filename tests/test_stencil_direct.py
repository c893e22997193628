"""The stencil without LDS: every tile at the edges of its lanes, rows and planes against the marching kernel, whose results
it repeats bit for bit, and the tables that the planner takes."""
import pytest

import paper_2405_05118_amd as mdh

torch = pytest.importorskip("torch")


def tables(shape):
    all_ = [mdh.mdh_candidate(mdh.MDH_STENCIL, shape, i) for i in range(mdh.mdh_num_candidates(mdh.MDH_STENCIL, shape))]
    return [p for p in all_ if p.in_region[0] == 2], [p for p in all_ if p.in_region[0] == 1]


def test_planner():
    direct, march = tables((100, 90, 200))
    assert {(p.prt[2][1], p.prt[2][0]) for p in direct} == {(2, 2), (2, 4), (4, 2), (4, 4), (1, 2), (2, 1)} and march
    assert mdh.mdh_default_params(mdh.MDH_STENCIL, (100, 90, 200)).in_region[0] == 2
    assert mdh.mdh_default_params(mdh.MDH_STENCIL, (512, 512, 512)).in_region[0] == 1
    for layer, d, v in ((0, 0, 2), (2, 0, 3), (2, 1, 3), (4, 1, 8), (5, 2, 32), (2, 0, (1 << 30) + 2)):
        q = direct[0].copy()
        q.ragged = 1
        q.prt[layer][d] = v
        assert mdh.mdh_validate_params(mdh.MDH_STENCIL, (100, 90, 200), q) != 0, (layer, d, v)


# the marching kernel where its workgroups are whole tiles and whole rounds of compute units
@pytest.mark.parametrize("shape,marches", [((512, 512, 512), True), ((256, 512, 512), True), ((512, 256, 512), True), ((256, 256, 1024), True), ((512, 544, 512), False),
                                           ((400, 400, 1024), False), ((512, 508, 512), False), ((512, 512, 500), False), ((200, 256, 512), False)])
def test_line_between_the_kernels(shape, marches):
    assert (mdh.mdh_default_params(mdh.MDH_STENCIL, shape).in_region[0] == 1) == marches


# grids of two or four planes, where both kernels have tiles of the same numbers: the marching one's is a candidate all the same
@pytest.mark.parametrize("shape,rows", [((2, 100, 200), 2), ((4, 40000, 128), 4)])
def test_marching_tables_are_offered(shape, rows):
    direct, march = tables(shape)
    same = [p for p in march if p.prt[0][0] == shape[0] and p.prt[2][1] == rows]
    assert any((p.prt[4][1] * p.prt[5][1], p.prt[4][2] * p.prt[5][2]) == (q.prt[4][1] * q.prt[5][1], q.prt[4][2] * q.prt[5][2]) and q.prt[2][:2] == [shape[0], rows]
               for p in same for q in [direct[0]]), [p.table() for p in same]


# a launch has less than 2^32 lanes: the longest grids stay with the kernel whose workgroups march over planes
@pytest.mark.parametrize("shape,marches", [((1 << 25, 1, 1), False), ((1 << 26, 1, 1), True), ((200000000, 1, 1), True), ((80000000, 2, 3), True), ((60000000, 3, 4), False)])
def test_grids_of_many_planes(shape, marches):
    p = mdh.mdh_default_params(mdh.MDH_STENCIL, shape)
    assert (p.in_region[0] == 1) == marches
    for q in [p] + sum(tables(shape), []):
        workgroups = q.prt[3][0] * q.prt[3][1] * q.prt[3][2]
        assert mdh.mdh_validate_params(mdh.MDH_STENCIL, shape, q) == 0 and (q.in_region[0] == 1 or workgroups * 256 < 1 << 32)
    if marches:
        q = tables((100, 1, 1))[0][0].copy()
        q.prt[3][0] = -(-shape[0] // q.prt[2][0])
        q.ragged = 1
        assert mdh.mdh_validate_params(mdh.MDH_STENCIL, shape, q) == 2  # MDH_ERR_SIZE


@pytest.mark.gpu
def test_a_grid_of_2_to_the_26_planes():
    n = 1 << 26
    x = torch.rand((n + 2, 3, 3), generator=torch.Generator(device="cuda").manual_seed(1), device="cuda")
    out = torch.full((n, 1, 1), float("nan"), device="cuda")
    mdh.mdh_stencil(x, out, 0.5, 1.0 / 12.0)
    c1 = float(torch.tensor(1.0 / 12.0))
    for a in range(0, n, 1 << 24):
        v = x[a : a + (1 << 24) + 2].double()
        m = v[1:-1]
        want = 0.5 * m[:, 1, 1] + c1 * (v[:-2, 1, 1] + v[2:, 1, 1] + m[:, 0, 1] + m[:, 2, 1] + m[:, 1, 0] + m[:, 1, 2])
        assert bool(((out[a : a + (1 << 24)].flatten().double() - want).abs() <= 7 * 2.0**-24 * want).all())  # as below


# one cell, one more and one less than the lanes' columns of each width, than their rows and planes; a last row and plane
# that end the buffer
@pytest.mark.gpu
@pytest.mark.parametrize("shape", [(1, 1, 1), (2, 3, 5), (5, 17, 63), (4, 33, 64), (3, 32, 65), (6, 31, 127), (7, 9, 129), (9, 16, 255), (8, 8, 257), (3, 65, 514)])
def test_same_as_the_marching_kernel(shape):
    g = torch.Generator(device="cuda").manual_seed(sum(shape))
    x = torch.rand([n + 2 for n in shape], generator=g, device="cuda")
    direct, march = tables(shape)
    n = shape[0] * shape[1] * shape[2]
    ref = torch.empty(shape, device="cuda")
    mdh.mdh_stencil(x, ref, 0.5, 1.0 / 12.0, march[0])
    v = x.double()
    c1 = float(torch.tensor(1.0 / 12.0))
    want = 0.5 * v[1:-1, 1:-1, 1:-1] + c1 * (v[:-2, 1:-1, 1:-1] + v[2:, 1:-1, 1:-1] + v[1:-1, :-2, 1:-1] + v[1:-1, 2:, 1:-1] + v[1:-1, 1:-1, :-2] + v[1:-1, 1:-1, 2:])
    assert bool(((ref.double() - want).abs() <= 7 * 2.0**-24 * want).all())  # seven roundings of positive terms
    for p in direct:
        guard = torch.full((n + 64,), 7.0, device="cuda")
        mdh.mdh_stencil(x, guard[:n].view(shape), 0.5, 1.0 / 12.0, p)
        assert torch.equal(guard[:n].view(shape), ref), p.table()
        assert bool((guard[n:] == 7.0).all())

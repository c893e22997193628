"""Record linkage with every number of fields: the loop of floating-point instructions against the definition, and its
hand-over to the integer loop at a record whose values it cannot hold."""
import numpy as np
import pytest

import oracle
import paper_2405_05118_amd as mdh

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nF", list(range(1, 17)))
@pytest.mark.parametrize("outside", ["none", "B", "A", "weights"])
def test_every_number_of_fields(nF, outside):
    rng = np.random.default_rng(100 + nF)
    nA, nB = 130, 4097
    A = rng.integers(0, 5, (nA, nF)).astype(np.int32)
    B = rng.integers(0, 5, (nB, nF)).astype(np.int32)
    wp = rng.integers(1, 1 << 16, nF).astype(np.int32)
    wm = rng.integers(-(1 << 16), 1, nF).astype(np.int32)
    if outside == "B":  # late in a part, in the middle of a block of four, and at both ends
        B[0, 0], B[2049, nF - 1], B[4096, 0] = -1, 1 << 23, np.iinfo(np.int32).min
        A[7, 0], A[8, nF - 1] = -1, 1 << 23
    elif outside == "A":
        A[3, 0] = -5
    elif outside == "weights":
        wp[0] = 1 << 24
    want_s, want_i = oracle.custom_reduce(A, B, wp, wm)
    dev = [torch.from_numpy(x).cuda() for x in (A, B, wp, wm)]
    s = torch.full((nA,), -7, dtype=torch.int32, device="cuda")
    i = torch.full((nA,), -7, dtype=torch.int32, device="cuda")
    n = mdh.mdh_workspace_size(mdh.MDH_CUSTOM_REDUCE, (nA, nB, nF))
    mdh.mdh_custom_reduce(*dev, s, i, None, torch.empty(n // 4, dtype=torch.int32, device="cuda") if n else None)
    assert np.array_equal(s.cpu().numpy(), want_s) and np.array_equal(i.cpu().numpy(), want_i)


# weights at the limits of what fp32 holds: their sum just below 2^24, the difference of a pair below, at and above 2^24
@pytest.mark.parametrize("nF", [1, 2, 8, 9, 16])
@pytest.mark.parametrize("pair", [((1 << 24) - 1, -((1 << 24) - 2)), ((1 << 23) + 1, -(1 << 23)), (1 << 23, -(1 << 23)),
                                  (-((1 << 24) - 1), (1 << 24) - 2)])
def test_weights_at_the_limit(nF, pair):
    rng = np.random.default_rng(nF)
    A = rng.integers(0, 2, (70, nF)).astype(np.int32)
    B = rng.integers(0, 2, (200, nF)).astype(np.int32)
    wp, wm = np.zeros(nF, np.int32), np.zeros(nF, np.int32)
    wp[nF - 1], wm[nF - 1] = pair
    B[:, nF - 1] = 2  # the last field agrees nowhere: every score holds w_disagree
    want_s, want_i = oracle.custom_reduce(A, B, wp, wm)
    dev = [torch.from_numpy(x).cuda() for x in (A, B, wp, wm)]
    s = torch.full((70,), -7, dtype=torch.int32, device="cuda")
    i = torch.full((70,), -7, dtype=torch.int32, device="cuda")
    n = mdh.mdh_workspace_size(mdh.MDH_CUSTOM_REDUCE, (70, 200, nF))
    mdh.mdh_custom_reduce(*dev, s, i, None, torch.empty(n // 4, dtype=torch.int32, device="cuda") if n else None)
    assert np.array_equal(s.cpu().numpy(), want_s) and np.array_equal(i.cpu().numpy(), want_i)

"""How the default scan cuts few long rows: a row that fits a workgroup's registers is not cut, a longer one into as many
tiles of 4096 a chunk as keep the chunks to a round of workgroups."""
import numpy as np
import pytest

import oracle
import paper_2405_05118_amd as mdh
from paper_2405_05118_amd import binding as B
from paper_2405_05118_amd import workloads as W

# rows, length, tiles a chunk, chunks a row
EDGES = [
    (1, 12289, 4, 1), (255, 16384, 4, 1), (1, 16385, 8, 1), (3, 32768, 8, 1), (3, 32769, 2, 5),
    (1, 128 * 8192, 2, 128), (1, 128 * 8192 + 1, 4, 65), (1, 256 * 16384, 4, 256), (1, 256 * 16384 + 1, 8, 129),
    (25, 40960, 2, 5), (26, 40960, 4, 3), (85, 40960, 4, 3), (86, 40960, 8, 2),
]


@pytest.mark.parametrize("R,n,tiles,chunks", EDGES)
def test_plan(R, n, tiles, chunks):
    p = mdh.mdh_default_params(mdh.MDH_SCAN, (R, n))
    assert (p.prt[B.L_VGPR][1], p.prt[B.L_WG][1], p.prt[B.L_WAVE][1]) == (4 * tiles, chunks, 16)
    words = 2 + R * chunks + R * ((chunks + 63) // 64) if chunks > 1 else 0
    assert mdh.mdh_workspace_size(mdh.MDH_SCAN, (R, n), p) == 8 * words


@pytest.mark.gpu
@pytest.mark.parametrize("R,n,tiles,chunks", EDGES)
def test_rows(R, n, tiles, chunks):
    """A lane adds up its four elements, a wavefront its lanes in six steps, and takes its own off again; the carries are fp64; one
    rounding when they become fp32, one in the last addition: 3 + 6 + 1 + 2 roundings, of sums of no more than the |x| up to
    the lane's last element."""
    import torch

    x = W.uniform(W.SEED_BASE + 97, 1, (R, n), -1, 1)
    ref, refabs = oracle.scan_rows(x, with_abs=True)
    nb = mdh.mdh_workspace_size(mdh.MDH_SCAN, (R, n))
    ws = torch.empty(nb // 4, device="cuda") if nb else None
    out = torch.full((R, n), float("nan"), device="cuda")
    mdh.mdh_scan(torch.from_numpy(x).cuda(), out, None, ws)
    bound = refabs[:, np.minimum(np.arange(n) | 3, n - 1)]
    assert float(np.max(np.abs(out.cpu().numpy() - ref) / bound)) <= 12 * 2.0**-24

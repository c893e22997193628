"""The walk over the records of B near the largest number of records: its bounds on the CPU, and one call there."""
import ctypes
import subprocess

import pytest

import paper_2405_05118_amd as mdh
from paper_2405_05118_amd.build import CSRC

torch = pytest.importorskip("torch")

WALK = r"""
#include "mdh_walk.h"
// walks [b0, b1) in runs and blocks of four as the kernel does; the number of records taken, or -1 where a position
// leaves [b0, b1 + 3] or a run is empty
extern "C" long long walk(int b0, int b1) {
  long long taken = 0;
  for (int done = b0; done < b1;) {
    const int end = mdh::run_end(done, b0, b1);
    if (end <= done || end > b1) return -1;
    for (long long bb = done; bb < end; bb += 4) {
      if (bb + 4 > 0x7fffffffll) return -1;
      for (int u = 0; u < 4; ++u) taken += bb + u < b1;
    }
    done = end;
  }
  return taken;
}
extern "C" long long most(void) { return mdh::kMaxWalked; }
"""


def test_bounds_of_the_walk(tmp_path):
    src, so = tmp_path / "walk.cpp", tmp_path / "walk.so"
    src.write_text(WALK)
    subprocess.check_call(["g++", "-O1", "-std=c++17", "-shared", "-fPIC", "-I", CSRC, str(src), "-o", str(so)])
    L = ctypes.CDLL(str(so))
    L.walk.restype = L.most.restype = ctypes.c_longlong
    most = L.most()
    # the last parts of a default call of the largest sizes, and parts of every length around a run
    for nB in (most, most - 1, 2**31 - 511, 2**31 - 512, 2**31 - 513, 2**31 - 1024, 2**30, 4097):
        chunk = -(-nB // 1024)
        for part in (0, 1, 1022, 1023):
            b0, b1 = min(part * chunk, nB), min((part + 1) * chunk, nB)
            assert L.walk(b0, b1) == b1 - b0, (nB, part)
    for n in (1, 3, 4, 31, 32, 33, 159, 160, 161, 511, 512, 513, 1025):
        assert L.walk(most - n, most) == n
        assert L.walk(7, 7 + n) == n


# one field, the most records that take the floating-point walk: the last run begins above 2^31 - 513
@pytest.mark.gpu
def test_most_records():
    nB = 0x7FFFFFF0
    B = torch.zeros((nB, 1), dtype=torch.int32, device="cuda")
    B[nB - 1], B[nB - 3], B[12345] = 3, 4, 5
    A = torch.tensor([[3], [4], [5], [0], [9]], dtype=torch.int32, device="cuda")
    wp = torch.tensor([7], dtype=torch.int32, device="cuda")
    wm = torch.tensor([-2], dtype=torch.int32, device="cuda")
    s = torch.empty(5, dtype=torch.int32, device="cuda")
    i = torch.empty(5, dtype=torch.int32, device="cuda")
    n = mdh.mdh_workspace_size(mdh.MDH_CUSTOM_REDUCE, (5, nB, 1))
    mdh.mdh_custom_reduce(A, B, wp, wm, s, i, None, torch.empty(n // 4, dtype=torch.int32, device="cuda"))
    assert s.tolist() == [7, 7, 7, 7, -2]
    assert i.tolist() == [nB - 1, nB - 3, 12345, 0, 0]

"""Custom reduce on bit maps: its grid and slots on the CPU, and its results where its parts meet, where scores tie and
where values or weights send it back to the loop over fields, against the definition."""
import ctypes
import subprocess

import numpy as np
import pytest

import oracle
import paper_2405_05118_amd as mdh
from paper_2405_05118_amd.build import CSRC

torch = pytest.importorskip("torch")

PLAN = r"""
#include "mdh_prl_bits.h"
using namespace mdh;
// 0 if the grid covers all records once, a queued pair fits its bits and two workgroups fit 160 KB of LDS
extern "C" int grid(long long nA, long long nB, int nF) {
  const PrlBitsGrid g = prl_bits_grid(nA, nB, nF);
  const long long c = (nB + kPrlChunk - 1) / kPrlChunk;
  if (g.sets < 1 || g.sets * 1024 > 1 << (32 - kPrlPartBits)) return 1;
  if ((long long)g.groups * g.sets * 1024 < nA || (long long)(g.groups - 1) * g.sets * 1024 >= nA) return 2;
  if ((long long)g.parts * g.chunks < c || (long long)(g.parts - 1) * g.chunks >= c) return 3;
  if ((long long)g.chunks * kPrlChunk > 1 << kPrlPartBits) return 4;
  if ((long long)g.groups * g.parts > 0x7fffffff) return 5;
  return 2 * prl_bits_lds_bytes(nF, g.sets) > 160 * 1024 ? 6 : 0;
}
// 0 if every field has 16 to 1024 slots, no two share one and all fit the maps
extern "C" int slots(const unsigned* used, int nF) {
  unsigned u[16];
  for (int f = 0; f < 16; ++f) u[f] = used[f];
  const PrlSlots s = prl_slots<16>(u, nF);
  for (int f = 0; f < nF; ++f)
    if (s.bits(f) < 4 || s.bits(f) > 10 || (f && s.first(f) != s.first(f - 1) + (1u << s.bits(f - 1)))) return 1;
  return s.first(nF - 1) + (1u << s.bits(nF - 1)) > kPrlMaps / 16 ? 2 : 0;
}
extern "C" int applies(int S, long long nA, long long nB, int nF) { return prl_bits_applies(S, nA, nB, nF); }
// bytes from the workspace to the word that tells whether the loop over fields had to do it
extern "C" long long stop(unsigned long long ws, long long nA, int S) { return (char*)&prl_bits_head((void*)ws, nA, S)->stop - (char*)ws; }
// bytes that keys, slots and head need, with 8 for alignment
extern "C" long long bytes(long long nA, int nF) { return 8 * nA + 4 * ((nF + 1) / 2) * nA + (long long)sizeof(PrlBitsHead) + 16; }
"""


@pytest.fixture(scope="module")
def plan(tmp_path_factory):
    d = tmp_path_factory.mktemp("bits")
    (d / "plan.cpp").write_text(PLAN)
    subprocess.check_call(["g++", "-O1", "-std=c++17", "-shared", "-fPIC", "-I", CSRC, str(d / "plan.cpp"), "-o", str(d / "plan.so")])
    L = ctypes.CDLL(str(d / "plan.so"))
    L.grid.argtypes = [ctypes.c_longlong, ctypes.c_longlong, ctypes.c_int]
    L.bytes.argtypes, L.bytes.restype = [ctypes.c_longlong, ctypes.c_int], ctypes.c_longlong
    L.stop.argtypes, L.stop.restype = [ctypes.c_ulonglong, ctypes.c_longlong, ctypes.c_int], ctypes.c_longlong
    L.applies.argtypes = [ctypes.c_int, ctypes.c_longlong, ctypes.c_longlong, ctypes.c_int]
    return L


def test_grid_slots_and_memory(plan):
    rng = np.random.default_rng(0)
    sizes = [(1024, 2**31 // 16, 16), (1024, 1, 1), (2**31 - 1, 1, 1), (1025, 129, 8), (1024, 2**31 - 1, 1), (65536, 2**18, 8)]
    sizes += [(int(2 ** rng.uniform(10, 20)), int(2 ** rng.uniform(0, 27)), int(rng.integers(1, 17))) for _ in range(3000)]
    for nA, nB, nF in sizes:
        assert plan.grid(nA, nB, nF) == 0, (nA, nB, nF)
        S = mdh.mdh_default_params(mdh.MDH_CUSTOM_REDUCE, (nA, nB)).prt[3][1]
        if plan.applies(S, nA, nB, nF):  # the head stays out of the first S - 1 parts' results
            assert plan.bytes(nA, nF) <= 8 * S * nA and 8 * nA >= 1200
            for ws in (1 << 20, (1 << 20) + 4):
                assert 8 * (S - 1) * nA <= plan.stop(ws, nA, S) <= 8 * S * nA - 1040 and (ws + plan.stop(ws, nA, S)) % 8 == 0
    for _ in range(2000):
        used = (rng.integers(0, 2**32, 16, dtype=np.uint64) >> rng.integers(0, 33, 16).astype(np.uint64)).astype(np.uint32)
        assert plan.slots(used.ctypes.data_as(ctypes.c_void_p), int(rng.integers(1, 17))) == 0


def check(plan, A, B, wp, wm, loop):
    """The result, and whether it is from the maps (loop = 0) or from the loop over fields (1; None: either)."""
    nA, nB, nF = len(A), len(B), A.shape[1]
    S = mdh.mdh_default_params(mdh.MDH_CUSTOM_REDUCE, (nA, nB)).prt[3][1]
    assert plan.applies(S, nA, nB, nF)
    want_s, want_i = oracle.custom_reduce(A, B, wp, wm)
    dev = [torch.from_numpy(np.ascontiguousarray(x)).cuda() for x in (A, B, wp, wm)]
    n = mdh.mdh_workspace_size(mdh.MDH_CUSTOM_REDUCE, (nA, nB, nF))
    ws = torch.empty(n // 4 + 1, dtype=torch.int32, device="cuda")
    for at in (0, 1):  # a workspace that is not aligned to more than its type, too
        s = torch.full((nA,), -7, dtype=torch.int32, device="cuda")
        i = torch.full((nA,), -7, dtype=torch.int32, device="cuda")
        mdh.mdh_custom_reduce(*dev, s, i, None, ws[at : at + n // 4])
        assert np.array_equal(s.cpu().numpy(), want_s) and np.array_equal(i.cpu().numpy(), want_i)
        if loop is not None:
            assert int(ws[at + plan.stop(ws[at:].data_ptr(), nA, S) // 4]) == loop


def inputs(nF, nA, top, seed, nB=None):
    rng = np.random.default_rng(seed)
    nB = nB or (1 << (29 if nF <= 10 else 31)) // (nF * nA) + 77
    A = rng.integers(0, top, (nA, nF)).astype(np.int32)
    B = rng.integers(0, top, (nB, nF)).astype(np.int32)
    return A, B, rng.integers(1, 1 << 16, nF).astype(np.int32), rng.integers(-(1 << 16), 1, nF).astype(np.int32)


# odd and even numbers of fields, one set of records of A and several, the last one nearly empty; 2 values: ties everywhere,
# in the same chunk, in other chunks and in other parts; 2^30: slots shared by different values
@pytest.mark.gpu
@pytest.mark.parametrize("nF,nA", [(1, 3137), (2, 40000), (3, 1024), (4, 5000), (7, 1025), (8, 4161), (9, 1100), (10, 2049),
                                   (11, 1500), (12, 3000), (13, 2100), (16, 4097)])
@pytest.mark.parametrize("top", [2, 60, 1 << 30])
def test_against_the_definition(plan, nF, nA, top):
    check(plan, *inputs(nF, nA, top, nF), loop=0 if top == 60 else None)


# agreeing never raises a score; it does in some fields; not at all; by steps no set of small weights follows; sums that
# wrap around, which the maps leave to the loop
@pytest.mark.gpu
@pytest.mark.parametrize("weights", ["lower", "mixed", "none", "steps", "wrap"])
def test_weights(plan, weights):
    A, B, wp, wm = inputs(8, 2300, 9, 5)
    if weights == "lower":
        wp, wm = wm, wp
    elif weights == "mixed":
        wp[::2], wm[::2] = wm[::2].copy(), wp[::2].copy()
    elif weights == "none":
        wp[:], wm[:] = 3, 3
    elif weights == "steps":
        wp[:], wm[:] = [10**k for k in (7, 6, 5, 4, 3, 2, 1, 0)], 0
    else:
        wp[:], wm[:] = 2**31 - 1, -(2**31)
    check(plan, A, B, wp, wm, loop=int(weights == "wrap"))


# every record of B is better than the one before, for all records of A: the most records that can be scored
@pytest.mark.gpu
def test_ever_better_records(plan):
    A, B, wp, wm = inputs(8, 1024, 60, 6)
    A[:] = 0
    B = B[np.argsort(np.where(B == 0, wp, wm).sum(axis=1), kind="stable")]
    check(plan, A, B, wp, wm, loop=None)


# More records to be scored than the maps are worth: values x + 2^9 x share one slot, so every record of B passes for every
# record of A.  In all of B: every workgroup gives up.  In the second half of B: some do, others are at work or done, and the
# loop over fields takes the place of their results.
@pytest.mark.gpu
@pytest.mark.parametrize("where", ["all", "half"])
@pytest.mark.parametrize("nF,nA", [(8, 2300), (7, 5000)])
def test_given_up_on_the_way(plan, nF, nA, where):
    A, B, wp, wm = inputs(nF, nA, 1 << 9, 7, 70001)  # parts of four to six chunks of 128
    other = np.maximum(B, 1)
    A += A << 9
    B += B << 9
    if where == "half":
        B[: len(B) // 2] = other[: len(B) // 2]
    check(plan, A, B, wp, wm, loop=1)


# The first record of B is the best but for few, so a bound that lets what is as good as it pass lets all of B pass: four sets
# of records of A, each with a first chunk to be scored, are no reason to give up.
@pytest.mark.gpu
def test_first_record_among_the_best(plan):
    rng = np.random.default_rng(8)
    A, B = (np.stack([rng.integers(0, a, n) for a in (4, 16, 64, 128)], 1).astype(np.int32) for n in (1 << 16, 1 << 17))
    wp, wm = rng.integers(-(1 << 16), 1, 4).astype(np.int32), rng.integers(1, 1 << 16, 4).astype(np.int32)
    check(plan, A, B, wp, wm, loop=0)


# captured, replayed on new records and weights with eager calls in between; the static scratch array's entry point too
@pytest.mark.gpu
def test_replays_and_static_scratch():
    nF, nA = 8, 2000
    sets = [inputs(nF, nA, top, 20 + top) for top in (3, 60, 7, 1 << 28)]
    nB = len(sets[0][1])
    dev = [torch.empty(n, dtype=torch.int32, device="cuda") for n in ((nA, nF), (nB, nF), (nF,), (nF,))]
    n = mdh.mdh_workspace_size(mdh.MDH_CUSTOM_REDUCE, (nA, nB, nF))
    ws = torch.empty(n // 4, dtype=torch.int32, device="cuda")
    out = [torch.empty(nA, dtype=torch.int32, device="cuda") for _ in range(4)]

    def fill(k):
        for d, x in zip(dev, sets[k]):
            d.copy_(torch.from_numpy(x))

    fill(0)
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        mdh.mdh_custom_reduce(*dev, out[0], out[1], None, ws)
    side.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=side):
        mdh.mdh_custom_reduce(*dev, out[0], out[1], None, ws)
    torch.cuda.synchronize()
    for k in (1, 2, 3, 0):
        fill(k)
        mdh.mdh_custom_reduce_static(*dev, out[2], out[3])
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        want = oracle.custom_reduce(*sets[k])
        for o, w in zip(out, want * 2):
            assert np.array_equal(o.cpu().numpy(), w), k

"""The plan of a paged GEMM call on the CPU: paths, workspace and forks as
functions of the layer's shape and the batch."""
import ctypes
import os

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
LIBP = os.path.join(os.path.dirname(HERE), "paper_2607_16184_amd", "libpw_hosttest.so")

DECODE, STREAM, TILED = range(3)
NO_LIMIT = (1 << 64) - 1


class Desc(ctypes.Structure):
    _fields_ = [(n, ctypes.c_int) for n in ("E", "H", "F", "R", "G", "act", "sdt")]


class Range:
    def __init__(self, v):
        self.ne, self.S, self.path, self.nsplit, self.kb, self.mtb, self.rt = v


class Plan:
    def __init__(self, E, K, H, F, T, n_shared=0, apl=False, n_16=0, n_pages=1, pages=0, ws=NO_LIMIT):
        if not os.path.exists(LIBP):
            from paper_2607_16184_amd import build
            build.build_hosttest()
        lib = ctypes.CDLL(LIBP)
        lib.pwt_gemm_plan.restype = None
        lib.pwt_gemm_plan.argtypes = ([ctypes.POINTER(Desc)] + [ctypes.c_int] * 4 + [ctypes.c_uint64] * 4
                                      + [ctypes.POINTER(ctypes.c_int64)])
        out = (ctypes.c_int64 * 18)()
        lib.pwt_gemm_plan(ctypes.byref(Desc(E, H, F, 64, 128, 1, 1)), T, K, int(apl), n_shared, n_16, n_pages, pages,
                          ws, out)
        self.total = out[0]
        self.routed, self.shared = Range(out[1:8]), Range(out[8:15])
        self.fork_shared, self.fork_shared_graph, self.fork_chains = (bool(v) for v in out[15:18])


@pytest.mark.parametrize("E,K,H,F,slots,path", [
    # gate/up tiles for at most half of the 256 CUs: the streaming kernel up to 127 slots ...
    (4, 1, 512, 512, 50, STREAM), (4, 1, 1024, 2048, 126, STREAM), (4, 2, 4096, 4096, 80, STREAM),
    (8, 2, 256, 512, 75, STREAM), (8, 2, 1024, 2048, 100, STREAM), (16, 2, 1024, 1024, 50, STREAM),
    (16, 2, 1024, 1024, 124, STREAM), (8, 2, 1024, 2048, 128, TILED), (4, 1, 512, 512, 128, TILED),
    # ... but for 16 or more experts of 65 to 120 slots and half the CUs ...
    (16, 2, 1024, 1024, 65, TILED), (32, 4, 1024, 512, 120, TILED), (32, 4, 1024, 384, 80, STREAM),
    # ... more than half the CUs, but 8 to 15 experts up to 56 slots or above 120
    (4, 2, 4096, 4608, 52, TILED), (8, 2, 4096, 2304, 56, STREAM), (8, 2, 4096, 2304, 57, TILED),
    (16, 2, 1024, 1152, 52, TILED), (8, 2, 3072, 3712, 75, TILED), (4, 2, 4096, 7168, 124, STREAM),
    (8, 2, 2048, 2304, 124, STREAM), (8, 2, 2048, 3072, 124, TILED), (16, 2, 1024, 1152, 124, TILED),
    # a tile for every CU
    (8, 2, 2048, 4096, 50, TILED), (8, 2, 4096, 14336, 75, TILED), (64, 6, 1024, 512, 124, TILED),
    # no 256-row down blocks
    (8, 2, 384, 4096, 80, STREAM), (8, 2, 384, 4096, 300, STREAM), (8, 2, 256, 512, 48, DECODE),
])
def test_path_of_the_routed_experts(E, K, H, F, slots, path):
    assert Plan(E, K, H, F, slots * E // K).routed.path == path


@pytest.mark.parametrize("E,K,H,F,slots,nsplit", [
    (8, 2, 2048, 4096, 80, 2), (8, 2, 4096, 7168, 80, 2), (32, 4, 1024, 1024, 80, 2), (16, 4, 1024, 2048, 80, 2),
    (64, 6, 1024, 768, 80, 1), (64, 6, 2048, 1408, 50, 1), (64, 6, 2048, 1408, 118, 1),     # more than half a round
    (64, 6, 1024, 512, 126, 1), (8, 2, 4096, 7168, 124, 2), (8, 2, 4096, 14336, 194, 2),     # 256-slot tiles
])
def test_down_splits_of_the_tiled_kernel(E, K, H, F, slots, nsplit):
    r = Plan(E, K, H, F, slots * E // K).routed
    assert r.path == TILED and r.nsplit == nsplit


@pytest.mark.parametrize("E,K,H,F,T,share16,rt", [
    (8, 2, 4096, 14336, 33, 0.0, 2), (8, 2, 4096, 14336, 33, 0.06, 1), (8, 2, 4096, 4096, 16, 0.1, 1),
    (8, 2, 4096, 4096, 16, 0.02, 2), (8, 2, 4096, 4096, 16, 0.03, 1),
    (8, 2, 4096, 4096, 4, 0.0, 1), (8, 2, 4096, 4096, 48, 0.0, 2), (64, 6, 2048, 1408, 33, 0.06, 2),
    (64, 6, 2048, 1408, 33, 0.07, 1), (64, 6, 1024, 1408, 33, 0.12, 2), (64, 6, 1024, 1408, 33, 0.13, 1),
    (8, 2, 4096, 14336, 64, 0.0, 2), (8, 2, 4096, 14336, 64, 0.12, 2), (8, 2, 4096, 14336, 64, 0.13, 1),   # two slot tiles
    (8, 2, 256, 512, 16, 0.0, 1),                                                      # too few workgroups
])
def test_row_tiles_of_the_decode_kernels(E, K, H, F, T, share16, rt):
    n = E * (2 * F + H) // 64
    r = Plan(E, K, H, F, T, n_16=int(share16 * n), n_pages=n).routed
    assert r.path == DECODE and r.mtb in (1, 2) and r.rt == rt


@pytest.mark.parametrize("E,n_shared,mib,T,eager,graph", [
    (64, 4, 48, 1, False, False), (64, 4, 48, 4, False, False), (64, 4, 48, 16, False, True),
    (64, 4, 48, 512, True, True), (64, 4, 96, 1, False, False), (64, 4, 96, 4, False, True),
    (64, 4, 96, 64, False, True), (64, 4, 96, 1024, True, True), (64, 4, 192, 256, True, True),
    (17, 1, 102, 1, False, True), (17, 1, 102, 64, True, True), (65, 1, 146, 16, False, True),
    (64, 4, 256, 1, True, True), (64, 0, 528, 64, False, False),
])
def test_fork_of_the_shared_experts(E, n_shared, mib, T, eager, graph):
    p = Plan(E, 4 + n_shared, 1024, 512, T, n_shared=n_shared, pages=mib << 20)
    assert (p.fork_shared, p.fork_shared_graph) == (eager, graph)


@pytest.mark.parametrize("E,K,mib,T,n_shared,fork", [
    (8, 2, 256, 16, 0, True), (8, 2, 255, 16, 0, False), (8, 2, 256, 3, 0, False), (8, 2, 256, 4, 0, True),
    (8, 2, 256, 200, 0, False), (10, 4, 256, 16, 2, False),
])
def test_fork_of_the_routed_chains(E, K, mib, T, n_shared, fork):
    assert Plan(E, K, 1024, 2048, T, n_shared=n_shared, pages=mib << 20).fork_chains == fork


def _one_copy(T, K, H, F):
    return T * K * (2 * F + 4 * H)


@pytest.mark.parametrize("E,K,H,F", [(64, 6, 2048, 1408), (32, 1, 4096, 128), (8, 2, 4096, 28672), (16, 4, 1024, 2048)])
def test_workspace_between_49_and_127_slots(E, K, H, F):
    """Every call of the range runs with one copy of the partials, so a
    workspace sized for more tokens always serves fewer; with room for two,
    the plan's split is used, whatever the static scratch holds."""
    lo, hi = -(-49 * E // K), 127 * E // K
    for T in range(lo, hi + 1, max(1, (hi - lo) // 97)):
        need = _one_copy(T, K, H, F)
        full = Plan(E, K, H, F, T)
        least = Plan(E, K, H, F, T, ws=need)
        if full.routed.path != TILED:
            continue
        assert least.total <= need + 512 and least.routed.nsplit == 1, T    # two 256-byte roundings
        assert Plan(E, K, H, F, T, ws=full.total).routed.nsplit == full.routed.nsplit
        if T + 1 <= hi:
            assert full.total <= Plan(E, K, H, F, T + 1).total, T


def test_workspace_from_128_slots_is_not_cut():
    """The two-copy need of larger batches stands: less is refused."""
    full = Plan(8, 2, 4096, 14336, 777)
    assert full.routed.path == TILED and full.routed.nsplit == 2
    assert Plan(8, 2, 4096, 14336, 777, ws=full.total - 1).total == full.total

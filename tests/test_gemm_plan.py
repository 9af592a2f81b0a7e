"""CPU checks of the W4A16 GEMM plans: workspace sizes, and the form that each
shape of the GPU tests takes."""
import ctypes
import os

import pytest


class Plan(ctypes.Structure):
    """ss::GemmPlan (ss_internal.h)."""
    _fields_ = [("nw", ctypes.c_int), ("nblocks", ctypes.c_int), ("nwg", ctypes.c_int), ("ksw", ctypes.c_int),
                ("knt", ctypes.c_int), ("wide", ctypes.c_bool), ("part_bytes", ctypes.c_size_t),
                ("prep_bytes", ctypes.c_size_t)]


@pytest.fixture(scope="module")
def ss():
    import paper_2506_11309_amd as ss
    if not os.path.exists(ss.LIB_PATH):
        import __graft_entry__
        __graft_entry__.build()
    ss.lib()
    return ss


@pytest.fixture(scope="module")
def plan(ss):
    """plan(M, K, N, swiglu): the library's own plan of a GEMM (an internal
    C++ function of the shared library)."""
    f = ctypes.CDLL(ss.LIB_PATH)["_ZN2ss15plan_w4a16_gemmEiiib"]
    f.restype = Plan
    f.argtypes = [ctypes.c_int, ctypes.c_int, ctypes.c_int, ctypes.c_bool]
    return f


# rows (every number of 16-row tiles, first and last), K and N over the range of the plan's lines
ROWS = (1, 8, 9, 16, 17, 32, 33, 48, 49, 64)
KS = tuple(range(128, 4096, 384)) + tuple(range(4096, 29000, 1536)) + (28672,)
NS = tuple(range(64, 2048, 192)) + tuple(range(2048, 36000, 1088)) + (36736,)


def test_plans_without_partials_ask_for_none(ss, plan):
    """K-split workgroups, and N-blocks that no two workgroups share, write no
    partial sums: the workspace holds the header and the prepared activations
    (as it did for SwiGLUs of many columns at up to 8 rows when they had
    K-split workgroups)."""
    assert ss.swiglu_workspace_bytes(8, 1024, 32960) == ss.WS_HEADER_BYTES + 16 * 1024 * 2
    seen = set()
    for swiglu in (False, True):
        size = ss.swiglu_workspace_bytes if swiglu else ss.gemm_workspace_bytes
        for K in KS:
            for N in NS:
                for M in ROWS:
                    p = plan(M, K, N, swiglu)
                    if not p.wide and (p.ksw or p.nblocks % p.nwg == 0):
                        seen.add((swiglu, p.ksw > 0))
                        assert size(M, K, N) == ss.WS_HEADER_BYTES + ss.prepared_bytes(M, K), (M, K, N, swiglu)
    assert seen == {(False, True), (True, True), (True, False)}


def test_size_queries_of_impossible_shapes_answer(ss):
    """Dimensions that the calls refuse (an empty FFN, fewer columns than a
    block) get a size from the queries, whatever the number of rows."""
    for T in (1, 17, 33, 64):
        for H, F in ((4096, 0), (4096, 32), (64, 4096), (0, 0)):
            assert ss.verify_layer_workspace_bytes(ss.make_dims(H, 32, 8, 128, F, 4096), T) >= ss.WS_HEADER_BYTES
        for K in (128, 4096, 16384, 28672):
            for N in (16, 48):
                assert ss.gemm_workspace_bytes(T, K, N) >= ss.WS_HEADER_BYTES
                assert ss.swiglu_workspace_bytes(T, K, N) >= ss.WS_HEADER_BYTES


def test_a_workspace_serves_fewer_rows(ss):
    """A workspace sized for some number of rows (tree nodes) is large enough
    for every smaller one, though the forms of fewer rows may write more
    partial sums and a smaller tree's attention may have more parts."""
    for size in (ss.gemm_workspace_bytes, ss.swiglu_workspace_bytes):
        for K in KS:
            for N in NS:
                sizes = [size(M, K, N) for M in ROWS]
                assert sizes == sorted(sizes), (size.__name__, K, N, sizes)
    for dims in ((8192, 16, 8, 128, 15232, 128), (2560, 16, 4, 64, 10752, 600), (8192, 64, 8, 128, 28672, 4160),
                 (4096, 32, 8, 128, 14336, 33000), (2048, 32, 8, 64, 8192, 640)):
        d = ss.make_dims(*dims)
        for size in (lambda T: ss.verify_layer_workspace_bytes(d, T), lambda T: ss.verify_step_workspace_bytes(d, T, 32000)):
            sizes = [size(T) for T in range(1, ss.MAX_TREE + 1)]
            assert sizes == sorted(sizes), dims

"""CPU checks of the W4A16 GEMM plans: workspace sizes, both sides of the plan's
lines, and the kernel instance that each shape of the GPU tests runs."""
import ctypes
import os
import sys

import pytest

sys.path.insert(0, os.path.dirname(os.path.abspath(__file__)))


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


@pytest.fixture(scope="module")
def norm(ss):
    """norm(plan, M, K, N, swiglu): whether the GEMM of that plan applies the
    RMSNorm of its input itself (the plan is then changed to that form's)."""
    f = ctypes.CDLL(ss.LIB_PATH)["_ZN2ss14norm_in_ksplitERNS_8GemmPlanEiiib"]
    f.restype = ctypes.c_bool
    f.argtypes = [ctypes.POINTER(Plan), ctypes.c_int, ctypes.c_int, ctypes.c_int, ctypes.c_bool]
    return lambda p, M, K, N, swiglu: f(ctypes.byref(p), M, K, N, swiglu)


# rows (every number of 16-row tiles, first and last), K and N over the range of the plan's lines
ROWS = (1, 8, 9, 16, 17, 32, 33, 48, 49, 64)
KS = tuple(range(128, 4096, 384)) + tuple(range(4096, 29000, 1536)) + (28672,)
NS = tuple(range(64, 2048, 192)) + tuple(range(2048, 36000, 1088)) + (36736,)


def test_plans_without_partials_ask_for_none(ss, plan):
    """K-split workgroups, and N-blocks that no two workgroups share, write no
    partial sums."""
    assert ss.swiglu_workspace_bytes(8, 1024, 32960) == ss.WS_HEADER_BYTES + 16 * 1024 * 2
    seen = set()
    for swiglu in (False, True):
        for K in KS:
            for N in NS:
                for M in ROWS:
                    p = plan(M, K, N, swiglu)
                    if not p.wide and (p.ksw or p.nblocks % p.nwg == 0):
                        seen.add((swiglu, p.ksw > 0))
                        assert p.part_bytes == 0, (M, K, N, swiglu)
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


def _form(p):
    return "wide" if p.wide else "K-split" if p.ksw else "stream-K"


# Both sides of the plan's lines, with the time of the K-split form over that
# of stream-K, weights from HBM.
@pytest.mark.parametrize("M,K,N,form", [
    # few columns, 17 rows and more, stream-K's blocks a multiple of 8: 1.02, 1.09; 0.93, 1.09; 0.91, 1.12
    (24, 8192, 1024, "K-split"), (24, 9216, 1024, "stream-K"), (46, 7168, 1024, "K-split"), (46, 9216, 1024, "stream-K"),
    (62, 6144, 1024, "K-split"), (62, 8192, 1024, "stream-K"),
    # 1.0, 1.08; 1.0, 1.12
    (24, 8192, 2048, "K-split"), (40, 8192, 1536, "stream-K"), (60, 6144, 2048, "K-split"), (60, 7168, 2048, "stream-K"),
    # not a multiple: 0.99, 1.11; 0.93, 1.05; 0.98, 1.13; 0.91, 1.04
    (30, 10240, 768, "K-split"), (30, 12288, 768, "stream-K"), (46, 10240, 1792, "K-split"), (46, 12288, 1792, "stream-K"),
    (62, 10240, 1792, "K-split"), (62, 12288, 1792, "stream-K"), (62, 10240, 1280, "K-split"), (62, 12288, 1280, "stream-K"),
    # few blocks: 0.98, 0.81; 0.92, 1.26; 0.94
    (62, 14336, 768, "K-split"), (40, 16384, 1024, "K-split"), (62, 20480, 1024, "K-split"), (62, 28672, 1024, "stream-K"),
    (40, 28672, 768, "K-split"),
    # 0.98, 1.04; 1.02, 1.12; 1.01; 1.02, 1.10
    (24, 10240, 4608, "K-split"), (24, 12288, 4608, "stream-K"), (40, 8192, 4608, "K-split"), (40, 10240, 4608, "stream-K"),
    (40, 10240, 6144, "K-split"), (46, 6144, 8448, "K-split"), (46, 8192, 8448, "stream-K"),
    # up to 16 rows: 0.98, 1.07; 0.95, 1.07; 1.0, 1.10; 0.95
    (16, 20480, 4608, "K-split"), (16, 28672, 4608, "stream-K"), (16, 12288, 8448, "K-split"), (16, 14336, 8448, "stream-K"),
    (16, 16384, 12288, "K-split"), (16, 20480, 12288, "stream-K"), (16, 28672, 14336, "K-split"),
    (24, 14336, 9216, "K-split"), (24, 16384, 9216, "wide"),
    # more than 1024 column tiles: 0.90, 1.27; 0.83, 1.04; 1.18; 0.96, 1.16; 1.08, 0.89
    (4, 7168, 16640, "K-split"), (4, 8192, 16640, "stream-K"), (4, 8192, 28992, "K-split"), (4, 8192, 28800, "stream-K"),
    (4, 8192, 35200, "stream-K"), (24, 4096, 28800, "K-split"), (46, 4096, 32768, "stream-K"),
    (24, 27008, 28800, "stream-K"), (24, 27008, 28992, "K-split"),
    # wide blocks at 17 to 32 rows: 0.90, 0.92; 0.84; 1.04
    (32, 28672, 8192, "wide"), (20, 20480, 8192, "wide"), (24, 16384, 8448, "stream-K"), (32, 18432, 8704, "wide"),
    (32, 18432, 6144, "stream-K"),
    # one K range of wide blocks at 17 to 32 rows 1.15 of stream-K, above 0.9
    (24, 12288, 32768, "wide"), (24, 12288, 36864, "stream-K"), (40, 12288, 49152, "wide")])
def test_plain_lines_with_weights_from_hbm(plan, M, K, N, form):
    assert _form(plan(M, K, N, False)) == form


@pytest.mark.parametrize("M,K,N,form", [
    # up to 32 rows: 1.0, 1.10 (also at 2 rows); 0.98
    (14, 20480, 6144, "K-split"), (14, 28672, 6144, "stream-K"), (2, 28672, 5120, "stream-K"), (8, 28672, 4096, "K-split"),
    (24, 20480, 1024, "K-split"), (24, 28672, 1024, "stream-K"),
    # above 32 rows: 0.95, 1.05; 1.12 at 60; 0.94, 1.13; up to 256 columns any K: 0.80; many columns too: 0.95
    (40, 10240, 2048, "K-split"), (40, 12288, 2048, "stream-K"), (60, 12288, 2048, "stream-K"),
    (40, 16384, 512, "K-split"), (60, 20480, 512, "stream-K"), (40, 28672, 256, "K-split"), (40, 28672, 7168, "K-split"),
    # two rounds of workgroups: 0.91, 1.07; 0.87, 1.10
    (24, 6144, 16384, "K-split"), (24, 6144, 17408, "stream-K"), (60, 3584, 9600, "K-split"), (60, 4096, 9600, "stream-K"),
    # more than 1088 column tiles, up to 8 rows: 0.80, 0.82; 0.89; 1.0
    (1, 3072, 17664, "K-split"), (8, 4096, 19200, "K-split"), (8, 1536, 24576, "K-split"), (8, 2048, 28672, "stream-K"),
    (8, 4224, 17664, "stream-K"), (9, 3072, 17664, "stream-K")])
def test_swiglu_lines_with_weights_from_hbm(plan, M, K, N, form):
    assert _form(plan(M, K, N, True)) == form


@pytest.mark.parametrize("K,N,waves,tiles", [
    (1024, 4096, 4, 2), (2048, 4096, 4, 2), (1280, 8192, 4, 4), (1536, 8192, 4, 4), (2048, 8192, 8, 4),
    (1280, 10240, 4, 2), (2048, 13312, 4, 2), (2048, 13376, 8, 4), (1536, 17408, 4, 4)])
def test_swiglu_with_norm_has_four_waves(plan, norm, K, N, waves, tiles):
    """The RMSNorm inside the SwiGLU: four waves where a workgroup's column is
    one tile (gate and up: 2) or K is at most 1536 (time over the present one
    with eight waves, weights from HBM, 8 rows: K 1280, N 2048 1.09, N 8192
    1.07, N 10240 1.17)."""
    for M in (1, 8, 16):
        p = plan(M, K, N, True)
        assert norm(p, M, K, N, True) and (p.ksw, p.knt) == (waves, tiles)


def test_norm_in_the_gemm_up_to_k_4096_for_few_rows(plan, norm):
    """Up to 8 rows and 256 column tiles the norm stays inside the GEMM up to
    K 4096 (K 3584, N 3712, 2 rows: the norm kernel 1.10 of its time)."""
    for M, K, N, inside in ((8, 4096, 4096, True), (1, 3584, 3712, True), (9, 2176, 4096, False), (8, 2176, 4160, False),
                            (8, 4224, 4096, False), (9, 2048, 4096, True)):
        assert norm(plan(M, K, N, False), M, K, N, False) == inside, (M, K, N)
    assert not norm(plan(8, 2176, 4096, True), 8, 2176, 4096, True)


def _instance(p, M, K, N, swiglu):
    """The kernel instance of plan p, and whether its blocks are split."""
    mt = (M + 15) // 16
    if p.wide:
        return "wide", mt, swiglu, p.nwg > p.nblocks
    if p.ksw:
        return "K-split", p.ksw, mt, p.knt, swiglu
    return "stream-K", mt, p.nw, swiglu, p.nblocks % p.nwg != 0


def _norm_instance(p, K, swiglu):
    groups = (4 if p.ksw == 4 and K > 1024 else 2) if swiglu else (4 if K > 2048 else 2)
    assert (K // 128 + p.ksw - 1) // p.ksw <= groups
    return "norm", p.ksw, p.knt, swiglu, groups


def _cases(test):
    """The shapes of a parametrised GPU test."""
    return [tuple(c) for m in test.pytestmark if m.name == "parametrize" for c in m.args[1]]


@pytest.fixture(scope="module")
def gpu_tests():
    import test_gpu_kernels
    return test_gpu_kernels


def test_gpu_tests_run_the_forms_they_name(plan, norm, gpu_tests):
    for test, form in ((gpu_tests.test_w4a16_k_split_forms, "K-split"), (gpu_tests.test_w4a16_wide_blocks, "wide"),
                       (gpu_tests.test_w4a16_stream_k_forms, "stream-K")):
        for c in _cases(test):
            assert _form(plan(*c)) == form, c
    split = [_instance(plan(*c), *c) for c in _cases(gpu_tests.test_w4a16_split_blocks_reuse_one_workspace)]
    assert all(i[-1] is True for i in split[3:]) and {i[0] for i in split} == {"K-split", "stream-K", "wide"}
    inside = [norm(plan(M, K, N, sw), M, K, N, sw)
              for M, K, N, ldx, sw in _cases(gpu_tests.test_rmsnorm_then_projection_matches_oracle)]
    assert inside == [True] * 15 + [False] * 8 + [True] * 7


def test_every_instance_the_plan_reaches_runs_in_a_gpu_test(plan, norm, gpu_tests):
    reached, tested = set(), set()
    for swiglu in (False, True):
        for K in KS + (1024, 1152, 1408, 1920, 2048, 2176, 16512, 20864):
            for N in NS + (1024, 4160, 6144, 8256, 16384, 17472, 32768):
                for M in ROWS:
                    p = plan(M, K, N, swiglu)
                    reached.add(_instance(p, M, K, N, swiglu))
                    if norm(p, M, K, N, swiglu):
                        reached.add(_norm_instance(p, K, swiglu))
    for test in (gpu_tests.test_w4a16_k_split_forms, gpu_tests.test_w4a16_wide_blocks, gpu_tests.test_w4a16_stream_k_forms):
        tested |= {_instance(plan(*c), *c) for c in _cases(test)}
    for M, K, N, ldx, swiglu in _cases(gpu_tests.test_rmsnorm_then_projection_matches_oracle):
        p = plan(M, K, N, swiglu)
        if norm(p, M, K, N, swiglu):
            tested.add(_norm_instance(p, K, swiglu))
    assert reached <= tested, sorted(map(str, reached - tested))
    assert len(reached) > 50

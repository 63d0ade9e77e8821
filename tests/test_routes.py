"""Which kernel the library's rules give a call (host only).

The GPU tests of a kernel name shapes that are meant to reach it.  The rules are
fitted to measured times and may be fitted again, so that a shape changes over
with every test still passing: here each list is held to the kernels and tiles
that it is meant for, at the 256 CUs of an MI355X.
"""

import os

import pytest

from paper_2609_33601_amd import jq
from tests.routes import few_rows, few_rows_batch, route

pytestmark = pytest.mark.skipif(not os.path.exists(jq.LIB_PATH),
                                reason="libjq.so not built (run __graft_entry__.build())")


def test_few_row_quantiser_only_where_it_is_faster():
    for G in (0, 64, 128):
        for K in (128, 3072, 12288, 16384):
            assert few_rows(1, K, G) and few_rows(512, K, G) and not few_rows(513, K, G)
    # longer rows: measured slower than the one-row kernel here
    for K in (20480, 49152, 65536):
        for M in (1, 192, 384, 512):
            assert not few_rows(M, K), (M, K)
        for M in (16, 64, 128, 256, 512):
            assert not few_rows(M, K, 64) and not few_rows(M, K, 128), (M, K)
        assert few_rows(64, K) and few_rows(2, K, 64) and few_rows(2, K, 128)


@pytest.mark.parametrize("shapes", [[(512, 4096)] * 2, [(512, 4096)] * 4, [(512, 16384)] * 2, [(256, 12288)] * 4,
                                    [(512, 3072)] * 8, [(256, 3072)] * 4, [(600, 64), (1, 64)]], ids=str)
def test_batches_that_the_four_row_kernel_does_faster(shapes):
    assert not few_rows_batch(shapes)


@pytest.mark.parametrize("shapes", [[(64, 4096), (64, 12288)], [(128, 4096)] * 8, [(384, 8192)] * 2, [(1, 64)],
                                    [(512, 256)] * 4, [(29, 8832), (28, 37568), (2, 384)]], ids=str)
def test_batches_that_the_few_row_kernel_does_faster(shapes):
    assert few_rows_batch(shapes)


def test_quantiser_shapes_reach_the_few_row_kernel():
    from tests.test_gpu_quant_few import test_few_rows_batch, test_few_rows_equal_many

    shapes = _params(test_few_rows_equal_many, "M,K")
    for G in (0, 64, 128):
        lengths = {K for M, K in shapes if (not G or K % G == 0) and few_rows(M, K, G)}
        assert min(lengths) <= 128 and max(lengths) == 65536 and any(16384 < K < 65536 for K in lengths), (G, lengths)
    batches = _params(test_few_rows_batch, "shapes")
    assert {few_rows_batch(b) for b in batches if max(M for M, _ in b) <= 512} == {False, True}


@pytest.mark.parametrize("kind,M,K,N", [("w4a4", 8283, 9472, 792), ("w4a4", 680, 9920, 11083),
                                        ("w158a4", 2093, 7872, 4160), ("w158a4", 7778, 7168, 1152),
                                        ("w158a4", 1618, 11328, 4928)], ids=str)
def test_few_tile_kernel_gives_way_to_the_six_bit_one(kind, M, K, N):
    # both beat the int8 kernel's estimate; measured 8 to 50% faster on the 6-bit one
    assert route(kind, M, K, N).kernel == "wide"


def test_packed_gemm_shapes_reach_their_kernel():
    from tests import test_gpu_gemm_narrow, test_gpu_gemm_tiled, test_gpu_gemm_wide

    for kind, tiled, wide in (("w4a4", test_gpu_gemm_tiled.INT4, test_gpu_gemm_wide.INT4),
                              ("w158a4", test_gpu_gemm_tiled.TERNARY, test_gpu_gemm_wide.TERNARY)):
        for height, M, K, N in tiled:
            assert route(kind, M, K, N)[::2] == ("tiled", height), (kind, M, K, N)
        for h in (112, 128):
            assert {K % 128 for height, _, K, _ in tiled if height == h} == {0, 64}
        for bands, M, K, N, _ in wide:
            # int4 shapes of one step are the int8 kernel's
            assert route(kind, M, K, N)[::2] == (("wide", 32 * bands) if K > 256 else ("tiled", 112)), (kind, M, K, N)
        narrow = [route(kind, M, K, N) for M, K, N, _ in test_gpu_gemm_narrow.SHAPES]
        assert [r.kernel for r in narrow] == ["narrow"] * (len(narrow) - 2) + ["tiled"] * 2
        assert {(r.rows, r.cols) for r in narrow[:-2]} == {(32, 32), (64, 64), (64, 96)}
    # the extreme codes at the longest K
    assert route("w4a4", 4096, 65536, 4096).kernel == "wide"


def test_bf6_gemm_shapes_reach_their_kernel():
    from tests import test_gpu_f6_narrow, test_gpu_f6_tiles

    for bands, M, K, N, _ in test_gpu_f6_tiles.SHAPES:
        assert route("f6", M, K, N)[::2] == ("tiled", 32 * bands), (M, K, N)
    got = [route("f6", M, K, N) for M, K, N, _ in test_gpu_f6_narrow.SHAPES]
    want = [(32, 32)] * 7 + [(32, 64)] + [(64, 64)] * 3 + [(64, 96)] * 2
    assert [(r.rows, r.cols) for r in got[:-3]] == want and {r.kernel for r in got[:-3]} == {"narrow"}
    assert {r.kernel for r in got[-3:]} == {"tiled"} and {r.rows == 128 for r in got[-3:]} == {False, True}


def test_group_gemm_shapes_reach_their_kernel():
    from tests import test_gpu_group_narrow, test_gpu_group_tiles

    for M, K, N, G, _ in test_gpu_group_tiles.SHAPES:
        assert route("group_f6", M, K, N, G).kernel == "tiled", (M, K, N, G)
    got = [(K, G, route("group_f6", M, K, N, G)) for M, K, N, G, _ in test_gpu_group_narrow.SHAPES]
    assert {(G, r.waves) for _, G, r in got if r.kernel == "narrow"} == {(64, 4), (64, 8), (128, 4), (128, 8)}
    assert any(K % 128 == 64 and r.kernel == "narrow" and r.waves == w for K, _, r in got for w in (4, 8))
    assert sum(r.kernel == "tiled" for _, _, r in got) >= 4


def test_one_step_of_k_stays_off_the_six_bit_packed_kernel():
    # its loads run two steps of 256 codes ahead, at most into the block's next tile
    for kind in ("w4a4", "w158a4"):
        for K in (64, 192, 256):
            for M in (600, 1147, 1183, 2068, 4608, 7654, 9216):
                for N in (1152, 4096, 8192, 8960, 12288):
                    assert route(kind, M, K, N).kernel != "wide", (kind, M, K, N)
    assert route("w4a4", 1147, 192, 8960).kernel == "tiled"


def _params(test, names):
    """The values that a test is parametrised with over `names`."""
    return next(m.args[1] for m in test.pytestmark if m.name == "parametrize" and m.args[0] == names)

"""The planner of the matrix product on the host: which kernel a shape takes,
and that the shapes of the GPU tests still reach the kernels that they are
there for."""
import pytest

from gemm_launches import FORMATS, launches
from test_gpu_gemm_ex import FEW_ROWS_TILES, SHORT_K


@pytest.mark.parametrize("M,N,K,tile", FEW_ROWS_TILES)
def test_few_rows_shapes_reach_their_tiles(M, N, K, tile):
    """The same tile for all operands (one order of the sums), with ragged
    edges in every direction."""
    assert [launches(f, M, N, K) for f in FORMATS] == ["ks " + tile] * 3
    bm, bn = map(int, tile.split("x"))
    assert M % bm and M > bm and N % bn and N > bn and K % 128


def test_every_few_rows_tile_has_a_shape():
    assert len({tile for *_, tile in FEW_ROWS_TILES}) == len(FEW_ROWS_TILES) == 15


@pytest.mark.parametrize("M,N,K", [(705, 2944, 2304), (261, 13309, 2208), (391, 12099, 6560), (518, 2961, 992)])
def test_few_rows_tiles_refused_where_bf16_weights_lose(M, N, K):
    """A few-rows tile is 1.3 to 1.5 times the time of the other launches there
    for bf16 weights, and level for packed ones."""
    for f in FORMATS:
        assert not launches(f, M, N, K).startswith("ks")


@pytest.mark.parametrize("M,N,K", [(77, 20480, 2560), (226, 2560, 10240), (16, 1152, 6912)])
def test_few_rows_tiles_taken(M, N, K):
    for f in FORMATS:
        assert launches(f, M, N, K).startswith("ks")


@pytest.mark.parametrize("M,N,K,tile", SHORT_K)
def test_short_k_takes_the_general_kernel(M, N, K, tile):
    """gemm_tile_kernel takes up to 1.5 times as long there."""
    assert [launches(f, M, N, K) for f in FORMATS] == ["general " + tile] * 3


@pytest.mark.parametrize("M,N,K", [(339, 4798, 128), (1266, 8017, 192), (384, 5631, 704)])
def test_other_tiles_and_longer_k_do_not(M, N, K):
    for f in FORMATS:
        assert launches(f, M, N, K).startswith("tile")

"""The planner of the matrix product on the host: which kernel a shape takes,
and that the shapes of the GPU tests still reach the kernels that they are
there for."""
import pytest

from gemm_launches import FORMATS, launches
from test_gpu_gemm_ex import FEW_ROWS_TILES, K_TAILS, LONG_K_SHAPES, SHORT_K, SPLIT_SHAPES, TILE_STEPS


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


def test_every_tile_has_shapes_of_odd_and_even_steps():
    """All ten tiles with each of the three operands, ragged in M and N, over
    2 D + 1 steps or more (D register sets: 4 of the 64 x 128 tile, else 2)."""
    seen = set()
    for M, N, K in TILE_STEPS:
        for f in FORMATS:
            tile = launches(f, M, N, K)
            assert tile.startswith("tile ") and "+" not in tile
            bm, bn = map(int, tile[5:].split("x"))
            assert M % bm and N % bn and N % 32
            assert K // 64 >= (9 if (bm, bn) == (64, 128) else 5)
            seen.add((f, tile, K // 64 % 2))
    assert len(seen) == 10 * 3 * 2


@pytest.mark.parametrize("M,N,K,text", K_TAILS)
def test_k_tails_reach_the_general_tiles(M, N, K, text):
    assert [launches(f, M, N, K) for f in FORMATS] == [text] * 3


def test_split_shapes_split():
    segments = set()
    for M, N, K, _ in SPLIT_SHAPES:
        texts = [launches(f, M, N, K, work=True) for f in FORMATS]
        assert all("split" in t for t in texts)
        segments.add((texts[1].split()[0], K % 64 == 0, M % 256 == 0))
    assert {(f"split{k}", whole, False) for k in (2, 3, 4) for whole in (False, True)} <= segments
    for M, N, K, _ in LONG_K_SHAPES:
        assert all("split" not in launches(f, M, N, K, work=True) for f in FORMATS)

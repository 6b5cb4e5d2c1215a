"""Kernel and stream of the bf16 expert networks: both sides of every limit of the rule."""
import pytest

import bench
from tests.ffn_choice import choose, dense_tile_rows, first_half_beside_route, second_half_workgroups

STREAMING, TILED = (False, False, False), (True, True, False)
BESIDE, BESIDE_TILED, BESIDE_STREAMING = (False, True, True), (True, True, True), (True, False, True)


@pytest.mark.parametrize("below,above,sizes", [
    # 4e8 weights: 9.4 rows an expert are tiled in a large layer only
    (STREAMING, (True, False, False), [(100, 1024, 64, 2034, 0, 600), (100, 1024, 64, 2035, 0, 600)]),
    # 40 GFLOP: the shared expert goes to its own stream
    (TILED, BESIDE_TILED, [(1000, 1024, 64, 1024, 1024, 5357), (1000, 1024, 64, 1024, 1024, 5358)]),
    # large: 8 rows an expert; 128 tokens
    (STREAMING, BESIDE_STREAMING, [(100, 2048, 64, 1408, 2816, 511), (100, 2048, 64, 1408, 2816, 512)]),
    (STREAMING, BESIDE, [(127, 2048, 64, 1408, 2816, 300), (128, 2048, 64, 1408, 2816, 300)]),
    # smaller: 10 rows an expert
    (STREAMING, TILED, [(200, 1472, 64, 1344, 0, 639), (200, 1472, 64, 1344, 0, 640)]),
    # 4.5 GFLOP below 48 rows an expert, 3 GFLOP from there
    (STREAMING, TILED, [(100, 1024, 8, 4096, 0, 178), (100, 1024, 8, 4096, 0, 179)]),
    (STREAMING, TILED, [(200, 1024, 4, 1024, 0, 476), (200, 1024, 4, 1024, 0, 477)]),
    (STREAMING, TILED, [(200, 1024, 8, 1536, 0, 383), (200, 1024, 8, 1536, 0, 384)]),
    # a wide shared expert over sparse experts: 7 GFLOP of its own; 128 tokens
    (STREAMING, TILED, [(278, 1024, 64, 256, 4096, 75), (279, 1024, 64, 256, 4096, 75)]),
    (STREAMING, TILED, [(127, 1024, 64, 256, 9024, 75), (128, 1024, 64, 256, 9024, 75)]),
    # 16 GFLOP, ten times the routed experts': its own stream, the routed experts tiled from 8 rows on
    (TILED, BESIDE, [(317, 1024, 64, 256, 8192, 75), (318, 1024, 64, 256, 8192, 75)]),
    (TILED, BESIDE_TILED, [(400, 1024, 64, 256, 8192, 1281), (400, 1024, 64, 256, 8192, 1280)]),
    (BESIDE, BESIDE_TILED, [(400, 1024, 64, 256, 8192, 511), (400, 1024, 64, 256, 8192, 512)]),
    # fewer than 160 tokens, more than half of the work: streaming
    (STREAMING, TILED, [(159, 1024, 8, 1024, 4096, 300), (160, 1024, 8, 1024, 4096, 300)]),
    (STREAMING, TILED, [(100, 1024, 8, 1024, 4096, 399), (100, 1024, 8, 1024, 4096, 400)]),
])
def test_both_sides_of_every_limit(below, above, sizes):
    assert [choose(*s) for s in sizes] == [below, above]


def test_a_layer_without_one_of_the_groups_has_one_stream():
    for T in (1, 40, 130, 1000, 16384):
        for Is, B in ((0, 6 * T), (0, T), (2816, 0), (45056, 0)):
            assert not choose(T, 2048, 64, 1408, Is, B)[2]
            assert not choose(T, 512, 16, 512, Is, B)[2]


@pytest.mark.parametrize("rows,col_tiles,most,height", [(1, 8, 64, 32), (256, 8, 64, 32), (257, 8, 64, 64), (512, 8, 64, 64),
                                                        (513, 8, 64, 96), (2048, 8, 64, 256), (100000, 8, 64, 256),
                                                        (33, 64, 64, 64), (33, 65, 64, 256)])
def test_height_of_dense_tiles(rows, col_tiles, most, height):
    assert dense_tile_rows(rows, col_tiles, most) == height


def test_second_half_ends_before_the_routed_experts():
    # 3.5 Is h / 16000 us against the routed weights at 6 TB/s: 59 and 92 us, 118 and 87, 118 and 173
    assert second_half_workgroups(600, 2048, 64, 1408, 2816, 1800, 1) == 64
    assert second_half_workgroups(600, 2048, 60, 1408, 5632, 1200, 1) == 128
    assert second_half_workgroups(600, 2048, 60, 1408, 5632, 1200, 2) == 64
    # few of the experts can have rows: 59 us against 2.9 an expert
    assert [second_half_workgroups(600, 2048, 64, 1408, 2816, b, 2) for b in (20, 21)] == [128, 64]


@pytest.mark.parametrize("T,d,Is,B,fp8,beside", [(16, 256, 2816, 48, False, True), (17, 256, 2816, 48, False, False),
                                                 (16, 255, 2816, 48, False, False), (16, 512, 2816, 48, True, True),
                                                 (16, 511, 2816, 48, True, False), (16, 2048, 8160, 48, False, True),
                                                 (16, 2048, 8192, 48, False, False), (1, 2048, 2816, 0, False, False),
                                                 (1, 2048, 0, 3, False, False)])
def test_shared_first_half_beside_the_routing(T, d, Is, B, fp8, beside):
    assert first_half_beside_route(T, d, 64, 1408, Is, B, fp8) == beside


def test_benchmark_counts_the_bytes_of_the_launch_it_times():
    """Decode shapes: the benchmark's own statement of the rule, for its count of the first half's bytes."""
    for T in (1, 8, 16, 17, 32):
        for d in (64, 192, 256, 448, 512, 2048):
            for Is in (0, 64, 2816, 8128, 8192, 22528):
                for B in (0, T, 4 * T):
                    for fp8 in (False, True):
                        if not any(choose(T, d, 64, 1408, Is, B)):
                            assert (bench.first_half_beside_route(T, d, Is, B, fp8) ==
                                    first_half_beside_route(T, d, 64, 1408, Is, B, fp8)), (T, d, Is, B, fp8)

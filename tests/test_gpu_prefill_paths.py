"""Both ways of the chunked prefill attention, at the edges of their tiles and splits.

Few query rows take the fused path (packed blocks reconstructed in LDS, the
key range split over workgroups when there are few query tiles), many rows the
workspace path (block images, 256-row tiles; 128 at D = 256 where tiles are
few).  Each case is checked against the fp64 oracle as in
test_gpu_prefill (2e-3 + 1e-2 |ref|), with lengths that leave a partial last
block, rows that leave a partial last tile, fp16 windows and sinks, rotation,
every code width and mixed widths, and asserts the path and the number of key
ranges that the dispatch rule gives it.
"""
import numpy as np
import pytest

from test_gpu_prefill import run

pytestmark = pytest.mark.gpu

NAMES = ["tiny_b16", "affine8", "sink64", "sym4_window", "kivi", "kivi_meta16", "hadamard", "perch_k4v2_window64",
         "kvarn_sink", "perch8_meta16", "gqa12b", "g256", "had_affine_window", "sym8_window_d256", "had8_d64", "had8_d128",
         "had8_d256", "had_perch_window"]


@pytest.mark.parametrize("name", NAMES)
def test_fused_key_ranges(name):
    # 1 unit, 46 rows, 47 blocks: one tile and eleven key ranges, the last block
    # partial (8-bit rotating codes at D = 256 do not fit the fused path's LDS)
    run(name, B=1, H=1, G=2, n=1493, C=23, seed=410, ranges=0 if name == "had8_d256" else 11)


@pytest.mark.parametrize("name,n,ranges", [("tiny_b16", 400, (1, 3)), ("kivi", 700, (5, 5)), ("gqa12b", 400, (3, 3))])
@pytest.mark.parametrize("C", [31, 32, 33, 64, 65])
def test_fused_tile_edges(name, n, ranges, C):
    # 4 C rows: 124 .. 260 on tiles of 128
    run(name, B=1, H=2, G=4, n=n + C, C=C, seed=420 + C, ranges=ranges[C >= 64])


@pytest.mark.parametrize("name", ["tiny_b16", "had_d64_g32"])
@pytest.mark.parametrize("shape", [dict(B=8, n=1001, C=65, ranges=4), dict(B=48, n=299, C=20, ranges=1)],
                         ids=["ranges", "one_range"])
def test_fused_two_workgroups_per_cu(name, shape):
    # head size 64: 128 tiles in four key ranges of eight blocks, the last
    # block partial, and 384 tiles of one range each
    run(name, H=8, G=2, seed=425, **shape)


@pytest.mark.parametrize("name", NAMES)
def test_workspace_tiles(name):
    # 32 units of 1 + 4 tiles of 256 rows: the workspace path at every head size
    run(name, B=4, H=8, G=4, n=293, C=260, seed=430, ranges=0)


D256 = ["gqa12b", "g256", "affine_g128_d256", "affine_g32_d256", "perch_d256", "had_affine_window", "sym8_window_d256",
        "had8_d256"]


@pytest.mark.parametrize("name", D256)
def test_workspace_few_tiles_d256(name):
    # 1040 rows per unit: nine tiles of 128, the last partial
    run(name, B=2, H=8, G=4, n=293, C=260, seed=440, ranges=0, tile_rows=128)


@pytest.mark.parametrize("name", D256)
def test_workspace_many_tiles_d256(name):
    # 320 rows per unit: 240 tiles of 256, half of them partial
    run(name, B=8, H=15, G=8, n=293, C=40, seed=445, ranges=0, tile_rows=256)


@pytest.mark.parametrize("name", ["tiny_b16", "kivi", "gqa12b", "hadamard"])
def test_split_outputs_do_not_depend_on_the_workspace(name):
    # 6 units in one pass, in groups of 4 + 2, and one at a time
    outs = [run(name, B=3, H=2, G=2, n=1100, C=30, seed=450, ws_units=u, ranges=8) for u in (None, 4, 1)]
    assert np.array_equal(outs[0], outs[1]) and np.array_equal(outs[0], outs[2])


@pytest.mark.parametrize("name", ["tiny_b16", "kivi", "hadamard", "gqa12b"])
def test_fused_calls_repeat_their_bits(name):
    # the outputs hold the first key range's partial sums until the merge
    outs = [run(name, B=1, H=2, G=2, n=1100, C=30, seed=455, ranges=8) for _ in range(4)]
    assert all(np.array_equal(outs[0], o) for o in outs[1:])

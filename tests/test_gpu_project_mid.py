"""The projection between the decode rows and the large prefill chunks.

Rows at the edges of the tiles, output widths that leave partial and
straddling column tiles (small shapes take 64x64 tiles, the larger ones assert
theirs), fewer K stages than the copy ring is deep,
and ranks that are not multiples of 16, against the fp64 oracle (2e-3 + 1e-2
|ref|, as in test_gpu_project).  Without an adapter every output is one chain
of products over K whichever kernel computes it, so a call's rows must equal
the same rows of a larger call bit for bit.
"""
import numpy as np
import pytest

import oracle

from gpu_util import assert_close, project_tile
from test_gpu_project import problem, run_gpu

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("M", [33, 63, 64, 65, 127, 129, 257])
@pytest.mark.parametrize("d_in,d_q,d_kv,r", [(64, 144, 48, 8), (192, 64, 16, 24), (320, 512, 272, 64)])
def test_mid_rows_match_oracle(M, d_in, d_q, d_kv, r):
    H, W, A, Bm = problem(500 + M + d_in, M, d_in, d_q, d_kv, r)
    y = run_gpu(H, W, A, Bm, r, 2.0, d_q, d_kv)
    ref, _ = oracle.project(H, W, A, Bm, r, 2.0, d_q, d_kv)
    assert_close(y, ref, what=f"M={M} d_in={d_in} d_q={d_q} d_kv={d_kv} r={r}")


# tiles: 0 128x128, 1 128x64, 2 64x64, -1 256x256
@pytest.mark.parametrize("tile,M,d_q,d_kv", [(1, 200, 3024, 576), (1, 250, 3024, 576), (0, 641, 4016, 752), (0, 765, 4016, 752)])
@pytest.mark.parametrize("r", [16, 24, 64])
def test_larger_tiles_match_oracle(tile, M, d_q, d_kv, r):
    # partial row and column tiles, and column tiles that straddle Q, K and V
    d_in = 128
    assert project_tile(M, d_q + 2 * d_kv) == tile
    H, W, A, Bm = problem(550 + M, M, d_in, d_q, d_kv, r)
    y = run_gpu(H, W, A, Bm, r, 2.0, d_q, d_kv)
    ref, _ = oracle.project(H, W, A, Bm, r, 2.0, d_q, d_kv)
    assert_close(y, ref, what=f"M={M} d_q={d_q} d_kv={d_kv} r={r}")


@pytest.mark.parametrize("tile,M", [(2, 40), (1, 200), (1, 400), (1, 900), (0, 641), (0, 700), (0, 768)])
def test_rows_do_not_depend_on_the_kernel(tile, M):
    # 64x64, 128x64 and 128x128 tiles at 6144 outputs against 256x256 tiles
    d_in, d_q, d_kv = 512, 4096, 1024
    assert project_tile(M, d_q + 2 * d_kv) == tile and project_tile(2304, d_q + 2 * d_kv) == -1
    H, W, A, Bm = problem(600, 2304, d_in, d_q, d_kv, 0)
    big = run_gpu(H, W, A, Bm, 0, 1.0, d_q, d_kv)
    assert np.array_equal(run_gpu(np.ascontiguousarray(H[:M]), W, A, Bm, 0, 1.0, d_q, d_kv), big[:M])


@pytest.mark.parametrize("M,r", [(1536, 64), (1552, 64), (4096, 48)])
def test_activation_pass_sizes(M, r):
    # 16x16 tiles, 64x48 tiles, and more than one round of those
    d_in, d_q, d_kv = 128, 64, 32
    H, W, A, Bm = problem(700 + r, M, d_in, d_q, d_kv, r)
    y = run_gpu(H, W, A, Bm, r, 2.0, d_q, d_kv)
    ref, _ = oracle.project(H, W, A, Bm, r, 2.0, d_q, d_kv)
    assert_close(y, ref, what=f"M={M} r={r}")

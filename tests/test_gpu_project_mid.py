"""The projection between the decode rows and the large prefill chunks.

Rows at the edges of the 64- and 128-row tiles, output widths that leave
partial and straddling column tiles, fewer K stages than the copy ring is deep,
and ranks that are not multiples of 16, against the fp64 oracle (2e-3 + 1e-2
|ref|, as in test_gpu_project).  Without an adapter every output is one chain
of products over K whichever kernel computes it, so a call's rows must equal
the same rows of a larger call bit for bit.
"""
import numpy as np
import pytest

import oracle

from gpu_util import assert_close
from test_gpu_project import problem, run_gpu

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("M", [33, 63, 64, 65, 127, 129, 257])
@pytest.mark.parametrize("d_in,d_q,d_kv,r", [(64, 144, 48, 8), (192, 64, 16, 24), (320, 512, 272, 64)])
def test_mid_rows_match_oracle(M, d_in, d_q, d_kv, r):
    H, W, A, Bm = problem(500 + M + d_in, M, d_in, d_q, d_kv, r)
    y = run_gpu(H, W, A, Bm, r, 2.0, d_q, d_kv)
    ref, _ = oracle.project(H, W, A, Bm, r, 2.0, d_q, d_kv)
    assert_close(y, ref, what=f"M={M} d_in={d_in} d_q={d_q} d_kv={d_kv} r={r}")


@pytest.mark.parametrize("M", [40, 200, 400, 900])
def test_rows_do_not_depend_on_the_kernel(M):
    # 64x64, 128x64 and 128x128 tiles at 6144 outputs against 256x256 tiles
    d_in, d_q, d_kv = 512, 4096, 1024
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

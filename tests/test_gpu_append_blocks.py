"""Whole, partial and mixed 32-token blocks in one append call, image bytes against the oracle.

The block coder writes whole blocks from registers and shared ones piece by
piece in the same launch; window and sink rows are moved several to a
workgroup.  Calls here start and end inside, at and around block boundaries
(heads, tails, both, neither), for every code width, mixed widths, per-channel
keys, rotation, windows, sinks and fp16 metadata.
"""
import pytest

from test_gpu_append import CASES, run_case

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("name", list(CASES))
@pytest.mark.parametrize("cuts", [(0, 200), (0, 5, 200), (0, 32, 33, 129, 160, 200), (0, 31, 95, 200)])
def test_block_edges(name, cuts):
    run_case(name, B=2, H=3, n=200, cuts=list(cuts), seed=800 + len(cuts))

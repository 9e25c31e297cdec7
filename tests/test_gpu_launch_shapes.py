"""Launch shapes of contexts that have tiles: the per-cell kernel keeps its own
range of jz chunks."""
import pytest

from test_gpu_mixed import prob
from test_gpu_tile import B  # noqa: F401

pytestmark = pytest.mark.gpu


def test_jz_chunks_of_the_per_cell_kernel(B):  # noqa: F811
    """957 cells of 8 planes: at most 8 jz chunks (one plane each), while the
    nine lane groups of a tile can be nine chunks."""
    C = B.Context(prob("cavity", nx=33, ny=29, nv=(24, 24, 8)), "fp32", tune="off")
    assert C.launch()["vsplit"] == 9
    for vec, unroll, persist in ((2, 1, 0), (4, 2, 0), (2, 3, 2)):
        C.set_launch(vec, unroll, 8, persist)
        with pytest.raises(B.BGKError) as e:
            C.set_launch(vec, unroll, 9, persist)
        assert e.value.code == B.E_INVALID
    C.set_launch(1, 1, 9, 0)
    with pytest.raises(B.BGKError):
        C.set_launch(1, 1, 10, 0)

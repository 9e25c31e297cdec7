"""Which streaming kernel a context runs (bgk_get_kernel): the tests of the
kernels on tiles reach them, and the cubes that no other test has on tiles --
plain upwind, Lie splitting, eight planes, a side too short for inner tiles.
Tolerances as in test_gpu_tile.py."""
import pytest

from test_gpu_mixed import prob
from test_gpu_tile import CUBES, FP32, FP64, MIXED, B, step_errors  # noqa: F401

pytestmark = pytest.mark.gpu

TILED = ([([prob(k, **o)], "fp64", "k_tile") for k, o in FP64] + [(MIXED, "fp64", "k_tile")] +
         [([prob(k, **o)], "fp32", "k_tile") for k, o in FP32] + [(CUBES[i], "fp32", "k_tile3") for i in (0, 1, 3)])


def test_kernel_of_each_form(B):  # noqa: F811
    for probs, prec, kernel in TILED:
        assert B.Context(probs, prec, tune="off").kernel() == kernel, (probs, prec)
    red = dict(reduced=True, vlo=(-4.0, -1.0, -1.0), vhi=(4.0, 1.0, 1.0))
    for cfg, prec, kernel in [(prob("cavity"), "fp32", "k_stream"), (prob("cavity3d", nx=16, ny=16, nz=16), "fp64", "k_stream"),
                              (prob("shock", nx=40, limiter="shift", splitting="lie", nv=(16, 16, 4)), "fp64", "k_shift"),
                              (prob("shock", nx=4500, limiter="shift", splitting="lie", nv=(16, 8, 16)), "fp64", "k_shift_rows"),
                              (prob("shock", nx=40, limiter="shift", splitting="lie", nv=(30, 1, 2), **red), "fp32",
                               "k_shift_cells")]:
        assert B.Context(cfg, prec, tune="off").kernel() == kernel, (cfg, prec)


@pytest.mark.parametrize("over", [dict(nx=20, ny=9, nz=28, nv=(26, 28, 8)), dict(nx=28, ny=20, nz=9, nv=(26, 28, 4), lid_mach=-0.2)])
def test_cubes_without_inner_tiles(B, oracle_mod, over):  # noqa: F811
    probs = [prob("cavity3d", splitting="lie", limiter="none", **over)]
    assert B.Context(probs, "fp32", tune="off").kernel() == "k_tile3"
    for v, i, ef, em in step_errors(B, oracle_mod, probs, "fp32", 3, (None, 3)):
        assert em <= 1e-5 and ef <= 1e-6, (v, i, ef, em)

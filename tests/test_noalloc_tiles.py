"""The allocation-free step on grids that run on tiles: the launch shape, and
with it every bit of f, is that of a fresh context, and tiles take no problem
beyond the static scratch array that fits it without them."""
import pytest
import torch

from paper_0903_4044_amd import binding, inputs
from test_gpu_mixed import prob

# 18000 cells with table entries of 53.8 MiB: partial sums for the 4 jz chunks
# of the per-cell kernel (6 MiB) fit the 64 MiB, for as many lane-group chunks
# as the tiles would take (16, 24 MiB) they do not
EDGE = prob("shock", nx=18000, nv=(128, 64, 2))


def test_tiles_leave_the_scratch_limit_alone():
    """A problem that fits gets as far as its NULL buffers."""
    L = binding.load()
    for nx, want in ((18000, binding.E_INVALID), (22000, binding.E_UNSUPPORTED)):
        arr = (binding.Problem * 1)(binding.to_struct(dict(EDGE, nx=nx)))
        assert L.bgk_step_noalloc(arr, 1, binding.FP32, None, None, 1, None, None) == want


@pytest.mark.gpu
@pytest.mark.parametrize("cfg,prec,chunks", [
    # more chunks than the per-cell kernel takes: 8 and 4
    (prob("cavity", nx=33, ny=29, nv=(24, 24, 8)), "fp32", 9), (prob("cavity", nx=24, ny=24, nv=(32, 32, 4)), "fp64", 8),
    (prob("cavity", nx=40, ny=40, nv=(32, 32, 4)), "fp32", None), (prob("shock", nx=1401, nv=(26, 28, 5)), "fp64", None),
    (prob("cavity3d", nx=15, ny=16, nz=14, nv=(32, 32, 4)), "fp32", None), (EDGE, "fp32", None)])
def test_noalloc_on_tiles_matches_a_context(cfg, prec, chunks):
    torch.cuda.set_device(0)
    C = binding.Context(cfg, prec, tune="off")
    assert C.kernel() in ("k_tile", "k_tile3") and chunks in (None, C.launch()["vsplit"])
    x = C.initial_state()
    g = torch.Generator(device="cuda").manual_seed(17)
    x *= 1 + 0.2 * (2 * torch.rand(C.f_elems, dtype=C.dtype, device="cuda", generator=g) - 1)
    for n in (1, 3):
        C.set_seed(0)
        ref = C.step(x, n=n)
        out, ws = torch.full_like(x, float("nan")), torch.empty_like(x)
        binding.step_noalloc(cfg, prec, x, out, n, ws)
        torch.cuda.synchronize()
        assert torch.equal(out, ref), n

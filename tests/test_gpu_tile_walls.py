"""Wall fluxes of the three-dimensional tile kernel (k_tile3): the densities
that the walls across z emit come from the half-range fluxes of v_z, one of
which is completed from two lanes' sums.

Cavities with a strong flow along z, so that the two half-range fluxes differ
by an order of magnitude and a wrong one shows in the emitted density at once.
The floating-point error of a step is that of test_gpu_tile.py: FP32 values
within 1e-6 of the largest after 3 steps (one rounding of 1.2e-7 and float
increments of a few 6e-8 each), moments within 1e-5.
"""
import numpy as np
import pytest
import torch

from test_gpu_mixed import prob, speed

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def B():
    from paper_0903_4044_amd import binding
    binding.load()
    return binding


def wind(O, cfg, u):
    """The gas at rest seen from a frame moving along z, with a ripple in x."""
    nv, lo, hi = cfg["nv"], cfg["vlo"], cfg["vhi"]
    vx, vy, vz = (lo[a] + (np.arange(nv[a]) + 0.5) * (hi[a] - lo[a]) / nv[a] for a in range(3))
    m = np.exp(-(vz[:, None, None] - u) ** 2 - vy[None, :, None] ** 2 - vx[None, None, :] ** 2) * np.pi ** -1.5
    ripple = 1 + 0.1 * np.cos(np.arange(O.ncell))
    return (ripple[:, None] * m.reshape(1, -1)).reshape(O.shape)


def check(B, oracle_mod, cfg, f0, n, chunks):
    O = oracle_mod.Oracle(cfg)
    f0 = wind(O, cfg, f0)
    ref = O.step(f0, n)
    assert np.isfinite(ref).all()
    rm = O.moments(ref)
    C = B.Context(cfg, "fp32", tune="off")
    assert C.kernel() == "k_tile3"
    x = torch.tensor(f0.reshape(-1), dtype=torch.float32, device="cuda")
    for v in chunks:
        if v is not None:
            C.set_launch(1, 1, v, 0)
        y = C.step(x, n=n)
        got = y.cpu().numpy().astype(np.float64).reshape(O.shape)
        m = C.moments(y).cpu().numpy()
        ef = np.max(np.abs(got - ref)) / np.max(np.abs(ref))
        em = max(np.max(np.abs(m[:, 0] / rm[:, 0] - 1)), np.max(np.abs(m[:, 4] / rm[:, 4] - 1)),
                 np.max(np.abs(m[:, 1:4] - rm[:, 1:4])) / max(speed(cfg), 1.0))
        assert ef <= 1e-6 and em <= 1e-5, (v, ef, em)


@pytest.mark.parametrize("u", [1.2, -1.2])
def test_flow_onto_the_z_walls(B, oracle_mod, u):
    cfg = prob("cavity3d", nx=16, ny=16, nz=15, nv=(32, 32, 8), lid_mach=0.3)
    check(B, oracle_mod, cfg, u, 3, (None, 1, 3))


@pytest.mark.parametrize("lo,hi,u", [((-3.0, -3.0, -4.0), (3.0, 3.0, -0.5), -2.0), ((-3.0, -3.0, 0.5), (3.0, 3.0, 4.0), 2.0),
                                     ((0.5, -3.0, -3.0), (4.0, 3.0, 3.0), 0.0), ((-3.0, -4.0, -3.0), (3.0, -0.5, 3.0), 0.0)])
def test_one_sided_boxes(B, oracle_mod, lo, hi, u):
    """Velocity boxes on one side of v = 0 along an axis: one half-range flux
    is the whole sum, the other is zero, and the wall that it feeds emits
    nothing."""
    cfg = prob("cavity3d", nx=16, ny=15, nz=16, nv=(32, 32, 4), vlo=lo, vhi=hi)
    check(B, oracle_mod, cfg, u, 3, (None, 1, 3))

"""The streaming kernels on tiles of cells (k_tile, k_tile3) at the edges of its tiles,
halos, lane groups and velocity chunks, against the FP64 oracle.

Grids large enough for the tile kernel (its rule counts tiles times groups of
64 (jx, jy)), with sides that are no multiples of the tile, (jx, jy) planes
that are no multiples of 64 lanes, odd and even N_vz.

Tolerances: FP64 every f value within 1e-12 of the largest (n steps add a few
dozen roundings of 1.1e-16 of sums over ~1e3 velocities); FP32 moments within
1e-5 (one unbiased rounding of 6e-8 per step, averaged over the velocities);
the reverse step within 1e-12 of its largest entry.  In 3D also every FP32 f
value within 1e-6 of the largest: 3 steps of one rounding (1.2e-7) and of float
increments of a few 6e-8 each.
"""
import numpy as np
import pytest
import torch

from paper_0903_4044_amd import inputs
from test_gpu_mixed import initial, prob, speed

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def B():
    from paper_0903_4044_amd import binding
    binding.load()
    return binding


FP64 = [("cavity", dict(nx=26, ny=25, nv=(12, 11, 5))),
        ("cavity", dict(nx=25, ny=26, nv=(12, 11, 4), splitting="lie", limiter="none", lid_mach=-0.3)),
        ("cavity", dict(nx=14, ny=57, nv=(14, 10, 2), vlo=(-3.0, -3.0, -1.0), vhi=(3.0, 3.0, 1.0), reduced=True)),
        ("cavity", dict(nx=33, ny=23, nv=(12, 11, 7), maxwellian="conservative")),
        ("periodic2d", dict(nx=27, ny=31, nv=(8, 9, 6))),
        ("shock", dict(nx=1361, nv=(26, 28, 5))), ("periodic1d", dict(nx=1363, nv=(26, 28, 4), limiter="none"))]
FP32 = [("cavity", dict(nx=30, ny=31, nv=(26, 28, 5))), ("periodic2d", dict(nx=33, ny=29, nv=(26, 28, 4))),
        ("shock", dict(nx=757, nv=(26, 28, 5))), ("periodic1d", dict(nx=753, nv=(28, 26, 4)))]
MIXED = [prob("shock", nx=11, nv=(12, 11, 4)), prob("cavity", nx=37, ny=41, nv=(12, 11, 4)),
         prob("periodic1d", nx=2, nv=(12, 11, 4)), prob("periodic2d", nx=2, ny=25, nv=(12, 11, 4)),
         prob("cavity", nx=25, ny=1, nv=(12, 11, 4))]


def step_errors(B, oracle_mod, probs, prec, n, chunks=(None,)):
    Os = [oracle_mod.Oracle(p) for p in probs]
    f0 = [initial(O, seed=80 + i) for i, O in enumerate(Os)]
    refs = [O.step(f, n) for O, f in zip(Os, f0)]
    C = B.Context(probs, prec, tune="off")
    assert C.launch()["vec"] == 1  # these even N_vx are 2 or 4 wide in the per-cell kernel
    x = torch.tensor(np.concatenate([f.reshape(-1) for f in f0]), dtype=C.dtype, device="cuda")
    for v in chunks:
        if v is not None:
            C.set_launch(1, 1, v, 0)
        y = C.step(x, n=n)
        torch.cuda.synchronize()
        mom = C.moments(y).cpu().numpy()
        for i, (O, ref) in enumerate(zip(Os, refs)):
            got = C.instance_view(y, i).cpu().numpy().astype(np.float64).reshape(O.shape)
            m, r = mom[C.cell_offsets[i]:C.cell_offsets[i] + O.ncell], O.moments(ref)
            em = max(np.max(np.abs(m[:, 0] - r[:, 0]) / r[:, 0]), np.max(np.abs(m[:, 4] - r[:, 4]) / r[:, 4]),
                     np.max(np.abs(m[:, 1:4] - r[:, 1:4])) / speed(probs[i]))
            yield v, i, np.max(np.abs(got - ref)) / np.max(np.abs(ref)), em


@pytest.mark.parametrize("probs", [[prob(k, **o)] for k, o in FP64] + [MIXED])
def test_tile_fp64(B, oracle_mod, probs):
    for v, i, ef, em in step_errors(B, oracle_mod, probs, "fp64", 3, (None, 1, 2, 3)):
        assert max(ef, em) <= 1e-12, (v, i, ef, em)


@pytest.mark.parametrize("kind,over", FP32)
def test_tile_fp32(B, oracle_mod, kind, over):
    for v, i, ef, em in step_errors(B, oracle_mod, [prob(kind, **over)], "fp32", 4, (None, 5)):
        assert em <= 1e-5, (v, i, ef, em)


CUBES = [[prob("cavity3d", nx=15, ny=16, nz=14, nv=(32, 32, 4), lid_mach=0.3)],
         [prob("periodic3d", nx=16, ny=15, nz=14, nv=(32, 31, 5))],
         [prob("cavity3d", nx=18, ny=9, nz=28, nv=(26, 28, 8), splitting="lie", limiter="none")],
         [prob("shock", nx=7, nv=(32, 32, 4)), prob("cavity3d", nx=16, ny=16, nz=15, nv=(32, 32, 4)),
          prob("cavity", nx=8, ny=8, nv=(32, 32, 4))]]


@pytest.mark.parametrize("probs", CUBES)
def test_tile_fp32_3d(B, oracle_mod, probs):
    """Inner tiles and tiles at walls and periodic faces, sides that are no
    multiples of 4, a batch with lower dimensions."""
    for v, i, ef, em in step_errors(B, oracle_mod, probs, "fp32", 3, (None, 3)):
        assert em <= 1e-5 and ef <= 1e-6, (v, i, ef, em)


@pytest.mark.parametrize("kind,over", [FP64[0], FP64[5]])
def test_tile_record(B, oracle_mod, kind, over):
    """The recording pass on tiles: the step, its branch record (through the
    reverse step) and the record's moment sums."""
    cfg = prob(kind, **over)
    O = oracle_mod.Oracle(cfg)
    C = B.Context(cfg, "fp64", tune="off")
    f0 = initial(O, seed=90)
    lam = inputs.uniform(O.shape, seed=91, lo=-1, hi=1)
    dev = lambda a: torch.tensor(a.reshape(-1), device="cuda")
    y, rec = C.step_record(dev(f0))
    got, grad = C.step_adjoint_record(dev(f0), rec, dev(lam))
    got2, grad2 = C.step_adjoint(dev(f0), dev(lam))
    ref, (lref, gref) = O.step(f0, 1), O.step_adjoint(f0, lam)
    assert np.max(np.abs(y.cpu().numpy().reshape(O.shape) - ref)) <= 1e-12 * np.max(np.abs(ref))
    for l, g in ((got, grad), (got2, grad2)):
        assert np.max(np.abs(l.cpu().numpy().reshape(O.shape) - lref)) <= 1e-12 * np.max(np.abs(lref))
        np.testing.assert_allclose(g.cpu().numpy()[0], gref, rtol=1e-11, atol=1e-18)

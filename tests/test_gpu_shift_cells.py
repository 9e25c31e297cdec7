"""The translation form on small planes (k_shift_cells: several cells per
wave) at the edges of its lane segments, against the FP64 oracle: planes of
less than, exactly and between 16, 32 and 64 values, every jz chunking, cell
counts that leave a workgroup part empty.  Tolerances as in test_gpu_shift.py:
FP64 1e-12 of the largest value, FP32 moments 1e-5 after 6 steps."""
import numpy as np
import pytest
import torch

from test_gpu_shift import B, dev, moment_rel, perturbed, small  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("kind,nx,nv,red", [
    ("shock", 37, (5, 3, 4), False), ("periodic1d", 3, (4, 4, 5), False), ("shock", 21, (17, 1, 2), True),
    ("shock", 1, (32, 1, 2), True), ("periodic1d", 19, (8, 4, 3), False), ("shock", 130, (11, 3, 6), False),
    ("periodic1d", 33, (16, 4, 2), False), ("shock", 30, (64, 1, 2), True)])
def test_small_planes(B, oracle_mod, kind, nx, nv, red):  # noqa: F811
    over = dict(nx=nx, nv=nv, cfl=4.4)
    if red:
        over.update(reduced=True, vlo=(-4.0, -1.0, -1.0), vhi=(5.0, 1.0, 1.0))
    cfg = small(kind, **over)
    O = oracle_mod.Oracle(cfg)
    f0 = perturbed(O, 77)
    ref = O.step(f0, 6)
    for prec, dt in (("fp64", torch.float64), ("fp32", torch.float32)):
        C = B.Context(cfg, prec, tune="off")
        for vsplit in range(1, nv[2] + 1):
            C.set_launch(1, 1, vsplit, 0)
            y = C.step(dev(f0, dt), n=6)
            if prec == "fp64":
                np.testing.assert_allclose(y.cpu().numpy().reshape(O.shape), ref, rtol=0, atol=1e-12 * np.abs(ref).max())
            else:
                en, eV, eT = moment_rel(C.moments(y).cpu().numpy(), O.moments(ref))
                assert max(en, eV, eT) <= 1e-5, (vsplit, en, eV, eT)

"""The kernels on tiles against the per-cell kernel of the same context, over
the forms that both take: one-sided and lopsided velocity boxes, reduced
spaces in one and two dimensions, both Maxwellian forms, every splitting and
limiter, batches of several dimensions, odd planes and sides.

The two sum a cell's moments in another order and contract products otherwise,
so FP64 agrees within 1e-12 of the largest value and FP32, which may round a
value the other way, within 1e-6."""
import numpy as np
import pytest
import torch

from paper_0903_4044_amd import inputs
from test_gpu_mixed import prob
from test_gpu_tile import B  # noqa: F401

pytestmark = pytest.mark.gpu

NEG, POS = dict(vlo=(-4.5, -4.0, -4.0), vhi=(-0.25, 4.0, 4.0)), dict(vlo=(-4.0, 0.25, -3.0), vhi=(4.0, 4.5, 4.0))
RED2 = dict(vlo=(-4.0, -3.0, -1.0), vhi=(4.0, 3.0, 1.0), reduced=True)
RED1 = dict(vlo=(-4.0, -1.0, -1.0), vhi=(5.0, 1.0, 1.0), reduced=True)
FORMS = [
    [prob("cavity", nx=47, ny=39, nv=(17, 20, 5), **NEG)], [prob("cavity", nx=37, ny=61, nv=(20, 17, 4), splitting="lie", **POS)],
    [prob("periodic2d", nx=46, ny=39, nv=(26, 20, 3), limiter="none", **NEG)],
    [prob("cavity", nx=55, ny=63, nv=(20, 17, 2), maxwellian="conservative", **RED2)],
    [prob("periodic2d", nx=61, ny=53, nv=(17, 20, 2), splitting="lie", limiter="none", **RED2)],
    [prob("shock", nx=9300, nv=(90, 1, 2), **RED1)], [prob("periodic1d", nx=9300, nv=(65, 1, 2), **RED1)],
    [prob("shock", nx=2900, nv=(17, 20, 7), maxwellian="conservative"), prob("periodic1d", nx=101, nv=(17, 20, 7), splitting="lie")],
    [prob("cavity", nx=95, ny=79, nv=(20, 26, 6)), prob("shock", nx=57, nv=(20, 26, 6), limiter="none"),
     prob("periodic2d", nx=5, ny=31, nv=(20, 26, 6), maxwellian="conservative"), prob("cavity", nx=1, ny=47, nv=(20, 26, 6))],
]
FORMS3 = [
    [prob("cavity3d", nx=23, ny=19, nz=15, nv=(20, 26, 4), maxwellian="conservative")],
    [prob("periodic3d", nx=23, ny=15, nz=15, nv=(26, 20, 5), splitting="lie", limiter="none")],
    [prob("cavity3d", nx=15, ny=15, nz=23, nv=(20, 26, 4), vlo=(-4.0, -4.0, -4.5), vhi=(4.0, 4.0, -0.25)),
     prob("periodic3d", nx=6, ny=7, nz=9, nv=(20, 26, 4), vlo=(-4.0, -4.0, -4.5), vhi=(4.0, 4.0, -0.25))],
    [prob("cavity3d", nx=19, ny=20, nz=23, nv=(26, 20, 8)), prob("cavity", nx=24, ny=13, nv=(26, 20, 8)),
     prob("shock", nx=50, nv=(26, 20, 8), splitting="lie")],
]


def state(C, cfg, seed):
    """A Maxwellian near the middle of the velocity box with 20% noise."""
    ax = [cfg["vlo"][a] + (np.arange(cfg["nv"][a]) + 0.5) * (cfg["vhi"][a] - cfg["vlo"][a]) / cfg["nv"][a] for a in range(3)]
    e = [np.exp(-(v - 0.45 * (cfg["vlo"][a] + cfg["vhi"][a])) ** 2) for a, v in enumerate(ax)]
    if cfg.get("reduced"):
        e[2] = np.array([1.0, 0.5 if cfg["nv"][1] > 1 else 1.0])
    m = (e[2][:, None, None] * e[1][None, :, None] * e[0][None, None, :]).reshape(-1)
    f = m[None, :] * (1 + 0.2 * inputs.uniform((C.ncells, C.nvel), seed=seed, lo=-1, hi=1))
    return torch.tensor(f.reshape(-1), dtype=C.dtype, device="cuda")


@pytest.mark.parametrize("probs,prec", [(p, q) for p in FORMS for q in ("fp64", "fp32")] + [(p, "fp32") for p in FORMS3])
def test_tiles_match_the_per_cell_kernel(B, probs, prec):  # noqa: F811
    C = B.Context(probs, prec, tune="off")
    assert C.kernel() in ("k_tile", "k_tile3")
    chunks = C.launch()["vsplit"]
    x = state(C, probs[0], seed=31)
    C.set_launch(1, 2, 1, 0)
    assert C.kernel() == "k_stream"
    C.set_seed(5)
    ref = C.step(x, n=3).double()
    for v in (chunks, 1, 2):
        C.set_launch(1, 1, v, 0)
        C.set_seed(5)
        y = C.step(x, n=3).double()
        for i in range(len(probs)):
            a, b = C.instance_view(y, i), C.instance_view(ref, i)
            assert float((a - b).abs().max()) <= (1e-12 if prec == "fp64" else 1e-6) * float(b.abs().max()), (v, i)

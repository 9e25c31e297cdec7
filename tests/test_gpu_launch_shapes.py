"""Launch shapes of contexts that have tiles: (1, 1, chunks, 0) is the kernel
on tiles, every other shape the per-cell kernel that it named before tiles,
with the per-cell kernel's own range of jz chunks.  Values agree between the
two within 1e-6 of the largest (as in test_gpu_tile_edges.py), FP64 within
1e-12."""
import pytest
import torch

from paper_0903_4044_amd import inputs
from test_gpu_mixed import prob
from test_gpu_tile import B  # noqa: F401

pytestmark = pytest.mark.gpu

CASES = [("cavity", dict(nx=33, ny=29, nv=(24, 24, 8)), "fp32", "k_tile"), ("cavity", dict(nx=26, ny=25, nv=(14, 11, 5)), "fp64", "k_tile"),
         ("shock", dict(nx=1401, nv=(26, 28, 5)), "fp32", "k_tile"), ("cavity3d", dict(nx=15, ny=16, nz=14, nv=(32, 32, 4)), "fp32", "k_tile3")]


@pytest.mark.parametrize("kind,over,prec,kernel", CASES)
def test_per_cell_kernel_on_contexts_with_tiles(B, kind, over, prec, kernel):  # noqa: F811
    C = B.Context(prob(kind, **over), prec, tune="off")
    d = C.launch()
    assert C.kernel() == kernel and (d["vec"], d["unroll"], d["persist"]) == (1, 1, 0)
    x = C.initial_state()
    x = x * (1 + 0.2 * torch.tensor(inputs.uniform((C.f_elems,), seed=5, lo=-1, hi=1), dtype=C.dtype, device="cuda"))
    C.set_seed(7)
    ref = C.step(x, n=2).double()
    tol = 1e-12 if prec == "fp64" else 1e-6
    for unroll, persist in ((2, 0), (1, 2), (2, 1)) + (() if kind == "cavity3d" else ((3, 0), (4, 2))):
        for vsplit in (1, 2):
            C.set_launch(1, unroll, vsplit, persist)
            assert C.kernel() == "k_stream"
            assert {k: v for k, v in C.launch().items() if k != "tuned_us"} == dict(vec=1, unroll=unroll, vsplit=vsplit, persist=persist)
            y = C.step(x, n=2).double()
            assert float((y - ref).abs().max()) <= tol * float(ref.abs().max()), (unroll, vsplit, persist)
    C.set_launch(1, 1, d["vsplit"], 0)
    C.set_seed(7)
    assert C.kernel() == kernel and torch.equal(C.step(x, n=2).double(), ref)


def test_jz_chunks_of_the_per_cell_kernel(B):  # noqa: F811
    """957 cells of 8 planes: at most 8 jz chunks (one plane each), while the
    nine lane groups of a tile can be nine chunks."""
    C = B.Context(prob("cavity", nx=33, ny=29, nv=(24, 24, 8)), "fp32", tune="off")
    assert C.launch()["vsplit"] == 9
    for vec, unroll, persist in ((2, 1, 0), (4, 2, 0), (1, 2, 0), (1, 1, 2)):
        C.set_launch(vec, unroll, 8, persist)
        with pytest.raises(B.BGKError) as e:
            C.set_launch(vec, unroll, 9, persist)
        assert e.value.code == B.E_INVALID
    C.set_launch(1, 1, 9, 0)
    with pytest.raises(B.BGKError):
        C.set_launch(1, 1, 10, 0)


def test_persistent_batch_is_persistent(B):  # noqa: F811
    """A batch whose default is the tile kernel takes a persistent grid of the
    per-cell kernel when asked for one."""
    C = B.Context([prob("cavity", nx=31, ny=29, nv=(26, 28, 4), kn=k) for k in (0.1, 0.4)], "fp32", tune="off")
    s = C.launch()
    assert C.kernel() == "k_tile"
    C.set_launch(s["vec"], s["unroll"], min(s["vsplit"], 4), 2)
    assert C.kernel() == "k_stream" and C.launch()["persist"] == 2


def test_tuner_gives_small_translation_planes_no_persistent_grid(B):  # noqa: F811
    """k_shift_cells launches a plain grid whatever persist says: the tuner
    neither times such shapes again nor reports one."""
    C = B.Context(prob("shock", nx=3000, limiter="shift", splitting="lie", nv=(30, 1, 2), reduced=True,
                       vlo=(-4.0, -1.0, -1.0), vhi=(4.0, 1.0, 1.0)), "fp32", tune="off")
    for _ in range(3):
        s = C.autotune(C.initial_state())
        assert C.kernel() == "k_shift_rows" or s["persist"] == 0


def test_entry_and_exit_passes_do_not_follow_the_tiles_chunks(B):  # noqa: F811
    """The initial state and the closing relaxation write no partial sums:
    neither depends on how many chunks the tiles leave."""
    C = B.Context(prob("cavity", nx=26, ny=25, nv=(14, 11, 5), maxwellian="conservative"), "fp64", tune="off")
    assert C.kernel() == "k_tile"
    ref = C.initial_state()
    y = C.step(ref, n=1)
    for v in (1, 2):
        C.set_launch(1, 1, v, 0)
        assert torch.equal(C.initial_state(), ref)
        assert float((C.step(ref, n=1) - y).abs().max()) <= 1e-12 * float(y.abs().max())


@pytest.mark.parametrize("nz,red", [(2, True), (4, False), (32, False)])
def test_chunks_where_planes_are_few(B, nz, red):  # noqa: F811
    """72 tiles of 16 lane groups on 256 compute units: three chunks in one
    round of workgroups, not fifteen in five rounds, whose set-up each round
    repeats."""
    over = dict(vlo=(-4.0, -4.0, -1.0), vhi=(4.0, 4.0, 1.0), reduced=True) if red else {}
    C = B.Context(prob("cavity", nx=48, ny=48, nv=(32, 32, nz), **over), "fp64", tune="off")
    assert C.kernel() == "k_tile" and C.launch()["vsplit"] == 3


def test_reverse_step_from_a_record_at_any_chunk_count(B):  # noqa: F811
    """A record's totals serve the reverse step as they are, whatever number
    of partial sums the tiles leave when it runs."""
    C = B.Context(prob("cavity", nx=26, ny=25, nv=(14, 11, 5)), "fp64", tune="off")
    x = C.initial_state()
    x = x * (1 + 0.2 * torch.tensor(inputs.uniform((C.f_elems,), seed=8, lo=-1, hi=1), device="cuda"))
    lam = torch.tensor(inputs.uniform((C.f_elems,), seed=9, lo=-1, hi=1), device="cuda")
    _, rec = C.step_record(x)
    ref, gref = C.step_adjoint_record(x, rec, lam)
    for v in (1, 2, 3):
        C.set_launch(1, 1, v, 0)
        got, g = C.step_adjoint_record(x, rec, lam)
        assert torch.equal(got, ref) and torch.equal(g, gref)

"""The tuned-shape table: entries reach contexts of the streaming form they
were timed on and no others."""
import pytest

from paper_0903_4044_amd import binding, inputs


def test_entries_name_their_form():
    for key, shape in binding.load_tuned().items():
        size, form = key.rsplit("/", 1)
        assert size.rsplit("/", 1)[1].startswith("cells<=") and form in binding.FORMS.values()
        if form == "shift":
            assert shape["vec"] == 1 and shape["unroll"] <= 2


def test_tuned_shape_by_form():
    tile, cell = dict(vec=1, unroll=1, vsplit=12, persist=0), dict(vec=4, unroll=1, vsplit=1, persist=0)
    table = {"k/tiles": tile, "k/cells": cell}
    assert binding.tuned_shape(table, "k", "tiles") is tile
    assert binding.tuned_shape(table, "k", "cells") is cell
    assert binding.tuned_shape(table, "k", "shift") is None
    # entries saved without a form: as before, but for the shape that tiles took over
    assert binding.tuned_shape({"k": cell}, "k", "cells") is cell
    for form in ("tiles", "cells", "shift"):
        assert binding.tuned_shape({"k": tile}, "k", form) is None
        assert binding.tuned_shape({"k": dict(tile, unroll=2)}, "k", form)["unroll"] == 2
        assert binding.tuned_shape({"k": dict(tile, persist=4)}, "k", form)["persist"] == 4


@pytest.mark.gpu
@pytest.mark.parametrize("cfg,prec,form,kernel,shape", [
    # translation: no entry at 48^3, its own default
    (dict(inputs.config("shock_m3_fp32"), nx=800, limiter="shift", splitting="lie"), "fp32", "shift", "k_shift_rows", None),
    # sides of 17 fail the padding rule of the tiles
    (inputs.config("cavity_64_adjoint", nx=17, ny=130), "fp32", "cells", "k_stream", (1, 2, 1, 0)),
    (inputs.config("cavity_64_adjoint"), "fp32", "tiles", "k_tile", (1, 1, 3, 0)),
    (inputs.config("shock_m3_fp32"), "fp32", "tiles", "k_tile", (1, 1, 12, 0))])
def test_contexts_take_their_form(cfg, prec, form, kernel, shape):
    C, D = binding.Context(cfg, prec), binding.Context(cfg, prec, tune="off")
    assert C.form == form and C.kernel() == kernel
    s = C.launch()
    got = (s["vec"], s["unroll"], s["vsplit"], s["persist"])
    d = D.launch()
    assert got == (shape or (d["vec"], d["unroll"], d["vsplit"], d["persist"]))

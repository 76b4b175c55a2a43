"""Layers that are not cut because only a reduction launch would add their sums: finished outputs (bias, scale, tanh) from
one chunk over all inputs, on every kernel that plans so, against the oracle; and that no such launch runs."""
import numpy as np
import pytest

from oracle import kan_oracle as ko
from paper_2512_15742_amd import synth

from kan_testlib import TOL_FP32, to_dev

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

TOL_HALF = 3e-3     # fp16 operands


# inputs that end inside a step, outputs that end inside a tile; the heads share their parameters (equal outputs)
@pytest.mark.parametrize("path,dims,heads,B", [
    ("precise", (17, 21), 1, 2), ("precise", (32, 1000), 1, 31), ("precise", (29, 130), 6, 16), ("precise", (82, 700), 70, 24),
    ("precise", (32, 333, 21), 1, 16),                                       # a middle layer: its successor takes no slices
    ("precise", (31, 3724), 7, 48), ("precise", (73, 1749), 21, 45), ("precise", (352, 2150), 12, 31),
    ("fp16", (23, 130), 1, 16), ("fp16", (30, 3297), 8, 10), ("fp16", (147, 866), 46, 36), ("fp16", (50, 571), 29, 37)])
@pytest.mark.parametrize("cb,gb", [("i8", "f16"), ("f32", "f32")])
def test_whole_layers(path, dims, heads, B, cb, gb):
    from paper_2512_15742_amd import binding as kb
    Ps = [synth.make_layer(8800 + 7 * l + dims[0], a, b, 1021, cb_dtype=cb, gb_dtype=gb) for l, (a, b) in enumerate(zip(dims, dims[1:]))]
    x = np.random.default_rng(B).uniform(-1.1, 1.1, size=(B, dims[0])).astype(np.float32)
    hs = [[kb.VQLayer(p) for p in Ps]] * heads
    p, tol = (kb.KAN_PATH_GATHER, TOL_FP32) if path == "precise" else (kb.KAN_PATH_MFMA, TOL_HALF)
    kb.kan_prof_begin(64)
    y = kb.kan_vq_head_forward(hs, to_dev(x), path=p)
    rec = kb.kan_prof_end()
    assert "kan_reduce@L1" not in rec, rec
    assert torch.equal(y, y[:1].expand_as(y))
    rep = ko.error_report(y[0].cpu().numpy(), ko.vq_head_forward(x, [q.as_dict() for q in Ps]))
    assert rep["headline"] <= tol * len(Ps), rep

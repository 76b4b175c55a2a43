"""Kernels on rotated basis words: the contraction that dequantises its own coefficients (kan_wide.hip): edges of its tiles of samples and outputs, odd and
ragged steps, every storage type, per-edge arrays that start anywhere, both rules, slices of a previous layer and
several heads, against the oracle; codebook rows that no edge uses.  The streaming contraction on tiles of 256 x 256
(kan_stream.hip): odd and ragged steps, tiles that the samples or outputs do not fill, chunks, slices, several heads."""
import dataclasses

import numpy as np
import pytest

from oracle import kan_oracle as ko
from paper_2512_15742_amd import synth

from kan_testlib import TOL_FP32, to_dev

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

TOL_HALF = 3e-3     # fp16 operands
TYPES = [("i8", "f16", "u16"), ("i8", "q8", "u16"), ("f32", "f32", "u16"), ("bfp8", "f16", "u16"), ("f16", "f32", "u32"),
         ("i8", "f32", "u32"), ("f32", "f16", "u16"), ("bfp8", "f32", "u32"), ("i8", "q8", "u32")]


@pytest.fixture(scope="module")
def kb():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2512_15742_amd import binding
    binding.lib()
    return binding


def shifted(kb, L, by):
    """The same layer with ids, gains and biases that start `by` elements into their allocations."""
    for name in ("idx", "gain", "bias"):
        t = getattr(L, name)
        buf = torch.zeros(t.numel() + by, dtype=t.dtype, device=t.device)
        buf[by:] = t.reshape(-1)
        setattr(L, name, buf[by:])
        setattr(L.desc, name, buf[by:].data_ptr())
    return L


def planned(kb, L, B, path):
    return kb.kan_vq_planned_kernel(L, B, 1, path)


def last_step_alone(P):
    """The layer with gain and bias 0 in all but the inputs of its last (ragged) step of 16: a result that lacks them is
    nothing like the right one, where among thousands of inputs they are within the fp16 bound."""
    kept = P.n_in - (P.n_in % 16 or 16)
    gain, bias = P.gain.copy(), P.bias.copy()
    gain[:kept], bias[:kept] = 0, 0
    return dataclasses.replace(P, gain=gain, bias=bias)


def check(y, x, P, tol, rows, rule="bspline"):
    assert np.isfinite(y).all()
    y_ref, A = ko.vq_layer_forward(x[rows], **P.as_dict(), rule=rule, return_abs=True)
    assert np.abs(y[rows] - y_ref).max() <= tol * max(np.abs(y_ref).max(), A.max())


@pytest.mark.parametrize("n_in,n_out,B,t", [
    (1033, 1021, 65, 0), (8300, 127, 128, 1), (2056, 512, 129, 2), (4097, 257, 256, 3), (1640, 640, 257, 4), (1033, 1021, 512, 5),
    (2056, 512, 600, 6), (16400, 64, 200, 7), (4100, 1030, 97, 8), (1033, 1025, 100, 0), (4100, 1030, 520, 1)])
def test_edges_of_tiles_and_steps(kb, n_in, n_out, B, t):
    cb, gb, idx = TYPES[t]
    P = synth.make_layer(9700 + n_in, n_in, n_out, 70000 if idx == "u32" else 4099, cb_dtype=cb, gb_dtype=gb, idx_dtype=idx)
    x = np.random.default_rng(B + n_in).uniform(-1.1, 1.1, size=(B, n_in)).astype(np.float32)
    x[0, 0], x[-1, -1] = 1.0, -1.0
    rows = np.unique(np.r_[0, 31, 32, 64, min(B, 128) - 1, B // 2, B - 1])
    tail = last_step_alone(P)
    for path, tol, name in ((kb.KAN_PATH_MFMA, TOL_HALF, "kan_wide" if (B, n_in) != (600, 2056) else "kan_mfma"),
                            (kb.KAN_PATH_GATHER, TOL_FP32, "kan_wide_split")):
        assert planned(kb, kb.VQLayer(P), B, path) == name
        y = kb.kan_vq_layer_forward(kb.VQLayer(P), to_dev(x), path=path)
        check(y.cpu().numpy(), x, P, tol, rows)
        check(kb.kan_vq_layer_forward(kb.VQLayer(tail), to_dev(x), path=path).cpu().numpy(), x, tail, tol, rows)
        for by in (1, 3):
            assert torch.equal(y, kb.kan_vq_layer_forward(shifted(kb, kb.VQLayer(P), by), to_dev(x), path=path))


def test_two_tap_rule(kb):
    P = synth.make_layer(9800, 1033, 1021, 4099, cb_dtype="i8", gb_dtype="f16")
    x = synth.make_x(9801, 130, 1033)
    for path, tol in ((kb.KAN_PATH_MFMA, TOL_HALF), (kb.KAN_PATH_GATHER, TOL_FP32)):
        y = kb.kan_vq_layer_forward(kb.VQLayer(P, rule=kb.KAN_RULE_PLI2), to_dev(x), path=path).cpu().numpy()
        check(y, x, P, tol, np.r_[0:4, 126:130], rule="pli")


@pytest.mark.parametrize("B", [70, 300])
def test_slices_and_heads(kb, B):
    """Two wide layers behind each other (the second adds the first one's slices) and a small last one, three heads."""
    dims = (700, 600, 620, 21)
    Ps = [[synth.make_layer(9900 + 10 * h + l, dims[l], dims[l + 1], 4099, cb_dtype="i8", gb_dtype="f16") for l in range(3)]
          for h in range(3)]
    x = synth.make_x(9901 + B, B, dims[0])
    hs = [[kb.VQLayer(p) for p in head] for head in Ps]
    for path, tol in ((kb.KAN_PATH_MFMA, TOL_HALF), (kb.KAN_PATH_GATHER, TOL_FP32)):
        kb.kan_prof_begin(64)
        y = kb.kan_vq_head_forward(hs, to_dev(x), path=path).cpu().numpy()
        rec = kb.kan_prof_end()
        assert "kan_prep_coef@L1" not in rec and "kan_prep_coef@L2" not in rec, rec       # no records are written
        name = "kan_wide" if path == kb.KAN_PATH_MFMA else "kan_wide_split"
        assert name + "@L1" in rec and name + "@L2" in rec and "kan_reduce@L1" not in rec, rec
        for h in range(3):
            rep = ko.error_report(y[h], ko.vq_head_forward(x, [p.as_dict() for p in Ps[h]]))
            assert rep["headline"] <= tol * 3, (path, h, rep)


def test_unused_codebook_rows_do_not_reach_the_result(kb):
    """Rows that no edge names may hold anything: tiles past the last column and steps past the last input fetch row 0
    or a row of an edge, never multiply the former."""
    P = synth.make_layer(9950, 1033, 1021, 4099, cb_dtype="f32", gb_dtype="f32")
    P.idx[P.idx == 0] = 1
    P.codebook[0] = np.nan
    x = synth.make_x(9951, 100, 1033)
    for path in (kb.KAN_PATH_MFMA, kb.KAN_PATH_GATHER):
        assert torch.isfinite(kb.kan_vq_layer_forward(kb.VQLayer(P), to_dev(x), path=path)).all()


@pytest.mark.parametrize("n_in,n_out,B,t", [(1033, 1021, 6100, 0), (4100, 1000, 1400, 2), (4111, 1023, 1300, 8), (333, 4095, 6200, 1),
                                            (6001, 1000, 2049, 3), (8200, 1000, 1100, 4), (2000, 2040, 3000, 5), (1000, 1000, 7000, 6),
                                            (1033, 1021, 6100, 7)])
def test_stream_edges_of_tiles_and_steps(kb, n_in, n_out, B, t):
    cb, gb, idx = TYPES[t]
    P = synth.make_layer(9600 + n_in, n_in, n_out, 70000 if idx == "u32" else 4099, cb_dtype=cb, gb_dtype=gb, idx_dtype=idx)
    x = np.random.default_rng(B + n_in).uniform(-1.1, 1.1, size=(B, n_in)).astype(np.float32)
    x[0, 0], x[-1, -1] = 1.0, -1.0
    rows = np.unique(np.r_[0, 31, 255, 256, B // 2, B - 1])
    tail = last_step_alone(P)
    for path, tol, name in ((kb.KAN_PATH_MFMA, TOL_HALF, "kan_stream"), (kb.KAN_PATH_GATHER, TOL_FP32, "kan_stream_split")):
        assert planned(kb, kb.VQLayer(P), B, path) == name
        for p in (P, tail):
            check(kb.kan_vq_layer_forward(kb.VQLayer(p), to_dev(x), path=path).cpu().numpy(), x, p, tol, rows)


@pytest.mark.parametrize("heads", [1, 3])
@pytest.mark.parametrize("dims,B,sliced", [((300, 1090, 1020, 40), 6100, False), ((3000, 1000, 3050, 40), 2100, True)])
def test_stream_slices_and_heads(kb, dims, B, sliced, heads):
    """Hidden rows of several heads; a layer that cuts its inputs into chunks in front, its slices added by the basis pass."""
    Ps = [[synth.make_layer(9650 + 10 * h + l, dims[l], dims[l + 1], 4099, cb_dtype="i8", gb_dtype="f16") for l in range(3)]
          for h in range(heads)]
    x = synth.make_x(9651, B, dims[0])
    hs = [[kb.VQLayer(p) for p in head] for head in Ps]
    rows = np.r_[0, 255, 256, B // 2, B - 1]
    ref = [ko.vq_head_forward(x[rows], [p.as_dict() for p in Ps[h]]) for h in range(heads)]
    for path, tol, name in ((kb.KAN_PATH_MFMA, TOL_HALF, "kan_stream"), (kb.KAN_PATH_GATHER, TOL_FP32, "kan_stream_split")):
        kb.kan_prof_begin(64)
        y = kb.kan_vq_head_forward(hs, to_dev(x), path=path).cpu().numpy()
        rec = kb.kan_prof_end()
        if sliced:      # the first layer by itself has slices to add
            kb.kan_prof_begin(64)
            kb.kan_vq_head_forward([h[:1] for h in hs], to_dev(x), path=path)
            assert "kan_reduce@L1" in kb.kan_prof_end()
        assert name + "@L2" in rec and (not sliced or name + "@L1" in rec) and "kan_reduce@L1" not in rec, rec
        for h in range(heads):
            rep = ko.error_report(y[h][rows], ref[h])
            assert np.isfinite(y).all() and rep["headline"] <= tol * 3, (path, h, rep)

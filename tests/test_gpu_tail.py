"""Matrix-core path, small layers in one launch (kan_tail.hip): steps per wave from none to several, ragged steps and
tiles, both tile widths, plain and sliced inputs with and without 16-byte loads, several heads, against the oracle."""
import numpy as np
import pytest

from oracle import kan_oracle as ko
from paper_2512_15742_amd import synth

from kan_testlib import TOL_FP32, to_dev

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

TOL_HALF = 3e-3     # fp16 operands
TYPES = [("i8", "f16", "u16"), ("i8", "q8", "u16"), ("f32", "f32", "u32"), ("bfp8", "f16", "u16")]


@pytest.fixture(scope="module")
def kb():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2512_15742_amd import binding
    binding.lib()
    return binding


def paths(kb):
    return (kb.KAN_PATH_MFMA, TOL_HALF), (kb.KAN_PATH_GATHER, TOL_FP32)


@pytest.mark.parametrize("n_in,n_out", [(1, 1), (15, 33), (16, 32), (17, 64), (63, 5), (127, 65), (128, 31), (130, 200), (257, 12),
                                        (446, 65), (448, 64)])
@pytest.mark.parametrize("B", [65, 96, 129, 4100])
def test_edges_of_steps_and_tiles(kb, n_in, n_out, B):
    cb, gb, idx = TYPES[(n_in + B) % len(TYPES)]
    P = synth.make_layer(9300 + n_in, n_in, n_out, 257, cb_dtype=cb, gb_dtype=gb, idx_dtype=idx)
    x = np.random.default_rng(B + n_in).uniform(-1.1, 1.1, size=(B, n_in)).astype(np.float32)
    rows = np.unique(np.r_[0:40, B // 2, B - 33:B])
    y_ref, A = ko.vq_layer_forward(x[rows], **P.as_dict(), return_abs=True)
    for path, tol in paths(kb):
        y = kb.kan_vq_layer_forward(kb.VQLayer(P), to_dev(x), path=path).cpu().numpy()
        assert np.isfinite(y).all()
        assert np.abs(y[rows] - y_ref).max() <= tol * max(np.abs(y_ref).max(), A.max()), (path, cb, gb, idx)


@pytest.mark.parametrize("dims", [(640, 132, 68, 5), (700, 131, 30), (96, 200, 37, 21, 3)], ids=lambda d: "-".join(map(str, d)))
@pytest.mark.parametrize("B,heads", [(65, 1), (300, 1), (97, 3)])
def test_slices_and_heads(kb, dims, B, heads):
    Ps = [[synth.make_layer(9400 + 10 * h + l, dims[l], dims[l + 1], 4099, cb_dtype="i8", gb_dtype="f16") for l in range(len(dims) - 1)]
          for h in range(heads)]
    x = synth.make_x(9500 + B, B, dims[0])
    hs = [[kb.VQLayer(p) for p in head] for head in Ps]
    for path, tol in paths(kb):
        y = kb.kan_vq_head_forward(hs, to_dev(x), path=path).cpu().numpy()
        for h in range(heads):
            rep = ko.error_report(y[h], ko.vq_head_forward(x, [p.as_dict() for p in Ps[h]]))
            assert rep["headline"] <= tol * (len(dims) - 1), (path, h, rep)


@pytest.mark.parametrize("hidden", [3, 61, 64, 65, 128, 129, 192, 193, 255, 256, 257, 333])
@pytest.mark.parametrize("n_in,B", [(1024, 97), (160, 66), (32, 70)])
def test_slices_of_every_width(kb, n_in, hidden, B):
    """A thread's share of a tile's inputs from one item of four to several, in many slices, few and none: the loads in flight
    differ."""
    Ps = [synth.make_layer(9700 + l, a, b, 701, cb_dtype="i8", gb_dtype="f32") for l, (a, b) in enumerate(((n_in, hidden), (hidden, 20)))]
    x = synth.make_x(9800 + hidden, B, n_in)
    head = [kb.VQLayer(p) for p in Ps]
    y_ref = ko.vq_head_forward(x, [p.as_dict() for p in Ps])
    for path, tol in paths(kb):
        y = kb.kan_vq_head_forward([head], to_dev(x), path=path)[0].cpu().numpy()
        rep = ko.error_report(y, y_ref)
        assert rep["headline"] <= 2 * tol, (path, rep)

"""Precise path, 2 to 32 samples, and fp16 path, up to 64: wave-by-wave kernel (kan_fused_wave.hip): loads of four edges at the ends of rows
and arrays, chunks of one to several groups of steps, both sample tiles, every storage width, against the oracle."""
import numpy as np
import pytest

from oracle import kan_oracle as ko
from paper_2512_15742_amd import synth

from kan_testlib import TOL_FP32, to_dev

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def kb():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2512_15742_amd import binding
    binding.lib()
    return binding


TYPES = [("i8", "f16", "u16"), ("i8", "q8", "u16"), ("i8", "f32", "u32"), ("f16", "f16", "u32"), ("f32", "f32", "u16"),
         ("bfp8", "f16", "u16")]


@pytest.mark.parametrize("n_in,n_out", [(1, 1), (3, 1), (1, 3), (1, 4), (2, 2), (5, 3), (17, 2), (16, 61), (31, 65), (48, 64),
                                        (65, 67), (130, 7), (1030, 5)])
@pytest.mark.parametrize("B", [2, 16, 17, 32])
def test_edges_of_rows_and_steps(kb, n_in, n_out, B):
    for n, (cb, gb, idx) in enumerate(TYPES):
        P = synth.make_layer(9000 + n, n_in, n_out, 257, cb_dtype=cb, gb_dtype=gb, idx_dtype=idx)
        x = np.random.default_rng(B + n_in).uniform(-1.1, 1.1, size=(B, n_in)).astype(np.float32)
        y_ref, A = ko.vq_layer_forward(x, **P.as_dict(), return_abs=True)
        y = kb.kan_vq_layer_forward(kb.VQLayer(P), to_dev(x), path=kb.KAN_PATH_GATHER).cpu().numpy()
        assert np.isfinite(y).all()
        assert np.abs(y - y_ref).max() <= TOL_FP32 * max(np.abs(y_ref).max(), A.max()), (cb, gb, idx)


@pytest.mark.parametrize("dims", [(2048, 64, 20), (1024, 36, 21), (640, 132, 68, 5)], ids=lambda d: "-".join(map(str, d)))
@pytest.mark.parametrize("B", [2, 13, 32])
def test_slices_into_the_next_layer(kb, dims, B):
    Ps = [synth.make_layer(9100 + l, dims[l], dims[l + 1], 4099, cb_dtype="i8", gb_dtype="f16") for l in range(len(dims) - 1)]
    x = synth.make_x(9200 + B, B, dims[0])
    y = kb.kan_vq_head_forward([[kb.VQLayer(p) for p in Ps]], to_dev(x), path=kb.KAN_PATH_GATHER)[0].cpu().numpy()
    rep = ko.error_report(y, ko.vq_head_forward(x, [p.as_dict() for p in Ps]))
    assert rep["headline"] <= TOL_FP32, rep


def test_call_that_fits_the_static_scratch_only_without_the_hand_over(kb):
    """64 heads whose partial sums fit the library's 32 MiB once: a reduction between the layers, right results."""
    B, dims, heads = 19, (36, 2992, 120, 184, 116), 64
    Ps = [synth.make_layer(9300 + l, dims[l], dims[l + 1], 4099, cb_dtype="i8", gb_dtype="f16") for l in range(len(dims) - 1)]
    head = [kb.VQLayer(p) for p in Ps]
    x = synth.make_x(9301, B, dims[0])
    y = kb.kan_vq_head_forward_static([head] * heads, to_dev(x), path=kb.KAN_PATH_GATHER)
    kb.kan_prof_begin(16)
    kb.kan_vq_head_forward_static([head] * heads, to_dev(x), path=kb.KAN_PATH_GATHER)
    assert "kan_reduce@L2" in kb.kan_prof_end()
    assert torch.equal(y, y[:1].expand_as(y))
    rep = ko.error_report(y[0].cpu().numpy(), ko.vq_head_forward(x, [p.as_dict() for p in Ps]))
    assert rep["headline"] <= TOL_FP32, rep


@pytest.mark.parametrize("dims,heads", [((64, 32, 8), 1),            # chunks of a single step, handed on and reduced
                                        ((2080, 40, 21), 1),         # more steps than slices may be handed on
                                        ((2048, 256, 21), 10),       # several workgroups per CU and several steps each
                                        ((333, 100, 10), 7)])
@pytest.mark.parametrize("B", [4, 16, 32])
def test_chunks_of_heads(kb, dims, heads, B):
    Ps = [[synth.make_layer(9400 + 3 * h + l, dims[l], dims[l + 1], 521, cb_dtype="i8", gb_dtype="f16") for l in range(2)]
          for h in range(heads)]
    x = synth.make_x(9500 + B, B, dims[0])
    y = kb.kan_vq_head_forward([[kb.VQLayer(p) for p in P] for P in Ps], to_dev(x), path=kb.KAN_PATH_GATHER).cpu().numpy()
    for h in (0, heads - 1):
        rep = ko.error_report(y[h], ko.vq_head_forward(x, [p.as_dict() for p in Ps[h]]))
        assert rep["headline"] <= TOL_FP32, rep


@pytest.mark.parametrize("rule", [0, 1], ids=["bspline", "pli"])
@pytest.mark.parametrize("n_in,n_out", [(1, 4), (5, 17), (16, 64), (17, 65), (49, 130), (300, 333)])
@pytest.mark.parametrize("B", [1, 15, 17, 33, 48, 49, 64])
def test_half_operands(kb, B, n_in, n_out, rule):
    """fp16 operands, blocks of 16 samples from one to four, every storage type: inputs that end inside a group of four and a
    step, outputs inside a lane's four and a tile.  Error per sample and output against the sum of |weight x coefficient|:
    weights, coefficients and gains are rounded to 2^-11 of themselves, an Int8 product once more."""
    for n, (cb, gb, idx, K) in enumerate((("i8", "f16", "u16", 4099), ("f32", "f32", "u32", 70001), ("f16", "f32", "u16", 300),
                                          ("i8", "q8", "u16", 65536), ("bfp8", "f16", "u16", 1000))):
        P = synth.make_layer(9600 + 10 * B + n, n_in, n_out, K, cb_dtype=cb, gb_dtype=gb, idx_dtype=idx)
        x = np.random.default_rng(B * 131 + n_in).uniform(-1.1, 1.1, size=(B, n_in)).astype(np.float32)
        x[0, 0], x[-1, -1] = -1.0, 1.0
        L = kb.VQLayer(P, rule=kb.KAN_RULE_PLI2 if rule else kb.KAN_RULE_BSPLINE3)
        assert kb.kan_vq_planned_kernel(L, B, 1, kb.KAN_PATH_MFMA) == "kan_fused_wave_f16"
        y = kb.kan_vq_layer_forward(L, to_dev(x), path=kb.KAN_PATH_MFMA).cpu().numpy()
        assert np.isfinite(y).all()
        name = "pli" if rule else "bspline"
        y_ref = ko.vq_layer_forward(x, **P.as_dict(), rule=name)
        coef = ko.reconstruct_coefficients(**P.as_dict())
        # (the biases are not rounded; shapes have mean 0, so a grid's mean is its bias and what is rounded is at most this)
        most = ko.dense_layer_forward(np.abs(coef) + np.abs(coef.mean(-1, keepdims=True)), x, rule=name)
        assert (np.abs(y - y_ref) <= 4 * 2.0 ** -11 * most + 1e-6 * np.abs(y_ref).max()).all(), (cb, gb, idx, ko.error_report(y, y_ref))


@pytest.mark.parametrize("B,dims,heads", [(37, (1000, 333, 21), 1), (64, (320, 96, 24), 20), (33, (70, 64, 32, 10), 3), (48, (128, 200, 17), 60)])
@pytest.mark.parametrize("cb,gb", [("i8", "f16"), ("f16", "f32")])
def test_half_operands_of_heads(kb, B, dims, heads, cb, gb):
    """Layers handed on in slices and reduced, several heads with parameters of their own."""
    n = min(heads, 3)
    Ps = [[synth.make_layer(9700 + 5 * h + l, a, b, 701, cb_dtype=cb, gb_dtype=gb) for l, (a, b) in enumerate(zip(dims, dims[1:]))] for h in range(n)]
    hs = [[kb.VQLayer(p) for p in P] for P in Ps]
    x = synth.make_x(9800 + B, B, dims[0])
    y = kb.kan_vq_head_forward([hs[h % n] for h in range(heads)], to_dev(x), path=kb.KAN_PATH_MFMA).cpu().numpy()
    for h in range(heads):
        assert np.array_equal(y[h], y[h % n])
    for h in range(n):
        rep = ko.error_report(y[h], ko.vq_head_forward(x, [p.as_dict() for p in Ps[h]]))
        assert rep["headline"] <= 3e-3 * len(dims), rep


@pytest.mark.parametrize("B,cb,gb,K", [(40, "f32", "f32", 65536), (64, "f32", "f16", 65536), (8, "f16", "f16", 45000)])
def test_one_large_codebook_at_a_time(kb, B, cb, gb, K):
    """Twenty heads whose codebooks do not fit an L2 beside each other: first layers in up to 64 workgroups each."""
    heads, dims = 20, (1003, 200, 21)
    Ps = [[synth.make_layer(9900 + 5 * h + l, a, b, K, cb_dtype=cb, gb_dtype=gb) for l, (a, b) in enumerate(zip(dims, dims[1:]))] for h in range(2)]
    hs = [[kb.VQLayer(p) for p in P] for P in Ps]
    x = synth.make_x(9950 + B, B, dims[0])
    y = kb.kan_vq_head_forward([hs[h % 2] for h in range(heads)], to_dev(x), path=kb.KAN_PATH_MFMA).cpu().numpy()
    for h in range(heads):
        assert np.array_equal(y[h], y[h % 2])
    for h in range(2):
        rep = ko.error_report(y[h], ko.vq_head_forward(x, [p.as_dict() for p in Ps[h]]))
        assert rep["headline"] <= 3e-3 * len(dims), rep

"""The precise path at batch 2..16 runs on tiles of 16 samples of the 16 x 16 x 4 fp32 matrix instruction: in the
wave-by-wave kernel, and for large layers and calls that fit the static scratch only so in the fused kernel (two blocks of 16 columns
per wave; tiles of 32 samples at batch 17..32).  Cases around that tile: batches that fill 1..4 of its
row groups or leave a ragged one, outputs that end inside either column block of a wave, inputs that end
inside a step and inside the pair of inputs a lane group serves; every storage type of ids, gains and rows
(the 16-byte metadata loads need outputs in multiples of 16, the others take the narrow loads)."""
import numpy as np
import pytest

from oracle import kan_oracle as ko
from paper_2512_15742_amd import synth

from kan_testlib import TOL_FP32, check_layer_output, to_dev

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def kb():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2512_15742_amd import binding
    binding.lib()
    return binding


SHAPES = [(9, 17), (70, 48), (33, 130), (257, 16), (64, 15), (16, 161)]


@pytest.mark.parametrize("B", [2, 6, 11, 15, 16, 17])
@pytest.mark.parametrize("shape", SHAPES, ids=lambda s: f"{s[0]}x{s[1]}")
def test_tile16_ragged(kb, B, shape):
    n_in, n_out = shape
    for n, (cb, gb, idx, K) in enumerate((("i8", "f16", "u16", 4099), ("f32", "f32", "u32", 70001), ("f16", "f16", "u16", 300),
                                          ("i8", "q8", "u16", 65536), ("bfp8", "f16", "u16", 1000))):
        P = synth.make_layer(7100 + 10 * B + n, n_in, n_out, K, cb_dtype=cb, gb_dtype=gb, idx_dtype=idx)
        x = np.random.default_rng(B * 131 + n_in).uniform(-1.1, 1.1, size=(B, n_in)).astype(np.float32)
        x[0, 0], x[-1, -1] = -1.0, 1.0
        L = kb.VQLayer(P)
        assert kb.kan_vq_planned_kernel(L, B, 1, kb.KAN_PATH_GATHER) == "kan_fused_wave"
        y_ref, A = ko.vq_layer_forward(x, **P.as_dict(), return_abs=True)
        y = kb.kan_vq_layer_forward(L, to_dev(x), path=kb.KAN_PATH_GATHER).cpu().numpy()
        rep = ko.error_report(y, y_ref, A)
        assert np.isfinite(y).all() and rep["headline"] <= TOL_FP32, (cb, gb, idx, rep)
        if n_in >= 8:
            assert rep["strict"] <= TOL_FP32, (cb, gb, idx, rep)


# one layer with two-byte gains, rows for 16-byte metadata loads and full tiles; the last step of 2101 inputs is cut short
@pytest.mark.parametrize("n_in,n_out,cb,idx,K,B", [(2101, 1648, "i8", "u32", 70001, 2), (2101, 1648, "i8", "u32", 70001, 16),
                                                   (2101, 1648, "bfp8", "u32", 70001, 32), (2600, 2688, "f16", "u16", 3000, 11),
                                                   (2600, 2688, "i8", "u16", 4099, 17)])
def test_large_layers_take_the_tiles_of_the_fused_kernel(kb, n_in, n_out, cb, idx, K, B):
    P = synth.make_layer(7400 + B, n_in, n_out, K, cb_dtype=cb, gb_dtype="f16", idx_dtype=idx)
    x = np.random.default_rng(B * 7 + n_in).uniform(-1.1, 1.1, size=(B, n_in)).astype(np.float32)
    L = kb.VQLayer(P)
    assert kb.kan_vq_planned_kernel(L, B, 1, kb.KAN_PATH_GATHER) == "kan_fused_f32"
    y = kb.kan_vq_layer_forward(L, to_dev(x), path=kb.KAN_PATH_GATHER).cpu().numpy()
    assert np.isfinite(y).all()
    check_layer_output(y, x, P, TOL_FP32, n_samples=96, full=False, seed=B)


# Every storage type: heads (which share their parameters: equal outputs) whose hidden activations leave the second layer's
# partial sums no room in the static scratch run the first on tiles.  Outputs that end inside either column block of a wave, inputs that
# end inside a step.
@pytest.mark.parametrize("dims,heads,B", [((29, 6328, 4), 60, 11), ((43, 4212, 21), 60, 16), ((51, 4034, 16), 60, 17), ((48, 2886, 4), 60, 24),
                                          ((61, 2060, 21), 60, 32)], ids=lambda v: str(v))
def test_calls_that_fit_the_static_scratch_only_on_tiles(kb, dims, heads, B):
    for n, (cb, gb, idx, K) in enumerate((("i8", "f16", "u16", 4099), ("f32", "f32", "u32", 70001), ("f16", "f16", "u16", 300),
                                          ("i8", "q8", "u16", 65536), ("bfp8", "f16", "u16", 1000))):
        Ps = [synth.make_layer(7500 + 3 * n + l, a, b, K, cb_dtype=cb, gb_dtype=gb, idx_dtype=idx) for l, (a, b) in enumerate(zip(dims, dims[1:]))]
        x = np.random.default_rng(B * 7 + dims[0]).uniform(-1.1, 1.1, size=(B, dims[0])).astype(np.float32)
        x[0, 0], x[-1, -1] = -1.0, 1.0
        hs = [[kb.VQLayer(p) for p in Ps]] * heads
        kb.kan_prof_begin(16)
        y = kb.kan_vq_head_forward_static(hs, to_dev(x), path=kb.KAN_PATH_GATHER)
        assert "kan_fused_f32@L1" in kb.kan_prof_end()
        assert torch.equal(y, y[:1].expand_as(y))
        rep = ko.error_report(y[0].cpu().numpy(), ko.vq_head_forward(x, [p.as_dict() for p in Ps]))
        assert rep["headline"] <= TOL_FP32, (cb, gb, idx, rep)


def test_tile16_matches_32_row_tile(kb):
    """The same rows through one block of 16 samples (batch 16) and two (batch 17, one more row): the same sums to
    fp32 rounding."""
    P = synth.make_layer(7300, 300, 200, 20001, cb_dtype="i8", gb_dtype="f16")
    x = synth.make_x(7301, 17, 300)
    L = kb.VQLayer(P)
    y16 = kb.kan_vq_layer_forward(L, to_dev(x[:16]), path=kb.KAN_PATH_GATHER).cpu().numpy()
    y17 = kb.kan_vq_layer_forward(L, to_dev(x), path=kb.KAN_PATH_GATHER).cpu().numpy()
    _, A = ko.vq_layer_forward(x[:16], **P.as_dict(), return_abs=True)
    assert (np.abs(y16 - y17[:16]) <= 2 * TOL_FP32 * A).all()

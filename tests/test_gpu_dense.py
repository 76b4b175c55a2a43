"""Dense baseline, one-pass kernels (kan_dense.hip): tiles of 16, 32 and 64 samples at the edges of
their tiles, against the oracle's dense layer."""
import numpy as np
import pytest

from oracle import kan_oracle as ko
from paper_2512_15742_amd import synth

from kan_testlib import TOL_FP32, check_dense_output, to_dev

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def kb():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2512_15742_amd import binding
    binding.lib()
    return binding


# (inputs: one, below / at / past a step of 16, of a wave group's 64 and of several chunks; outputs: one, tiles of
# 16 and 64 and one past them; batches: every tile, full and one past, two tiles of 64 and the last of the rule)
@pytest.mark.parametrize("n_in,n_out,B", [(1, 1, 1), (15, 16, 2), (16, 17, 16), (65, 15, 7), (129, 33, 16), (2050, 48, 9),
                                          (1, 1, 17), (17, 63, 32), (32, 64, 33), (33, 65, 64), (130, 129, 65),
                                          (300, 70, 128), (97, 40, 129), (64, 20, 256), (384, 2880, 39), (1408, 750, 18)])
def test_one_pass_kernels(kb, n_in, n_out, B):
    rng = np.random.default_rng(n_in * 7 + n_out + B)
    coef = (rng.standard_normal((n_in, n_out, 10)) * rng.uniform(1e-3, 2.0, (n_in, n_out, 1))).astype(np.float32)
    x = synth.make_x(B, B, n_in)
    x[0, 0], x[-1, -1] = 1.0, -1.0
    x[B // 2, n_in // 2] = np.float32(1.0 / 7.0)          # beside a knot
    y = kb.kan_dense_layer_forward(to_dev(coef), to_dev(x)).cpu().numpy()
    check_dense_output(y, x, coef, TOL_FP32)


@pytest.mark.parametrize("n_in,n_out,B", [(1033, 1021, 65), (2056, 512, 129), (4097, 257, 128), (1640, 640, 257), (300, 1090, 300), (520, 511, 1023),
                                          (1024, 256, 257), (500, 96, 1400),                # the contraction that converts its own coefficients
                                          (1024, 256, 256), (300, 64, 1024), (31, 33, 700),  # the last of the one-pass rule, many tiles of it
                                          (9000, 40, 128), (9000, 33, 200), (2784, 88, 194),  # tiles of 64 outputs half empty, or nearly: one pass
                                          (64, 2347, 253), (64, 1090, 505), (384, 2880, 65),  # whole, in one round of workgroups and in two
                                          (192, 64, 4979), (256, 4096, 1030)])                # many samples: the contraction again, records
def test_beyond_one_tile(kb, n_in, n_out, B):
    rng = np.random.default_rng(n_in + 3 * n_out + B)
    coef = (rng.standard_normal((n_in, n_out, 10)) * rng.uniform(1e-3, 2.0, (n_in, n_out, 1))).astype(np.float32)
    tail = coef.copy()
    tail[:n_in - (n_in % 16 or 16)] = 0                # the last step of 16 inputs alone
    x = synth.make_x(B, B, n_in)
    x[0, 0], x[-1, -1] = 1.0, -1.0
    rows = np.unique(np.r_[0, 31, 63, 64, min(127, B - 1), B // 2, B - 1])
    check_dense_output(kb.kan_dense_layer_forward(to_dev(coef), to_dev(x)).cpu().numpy()[rows], x[rows], coef, TOL_FP32)
    # (one edge's sum of four products can cancel to nothing: errors against the largest result, not against its |phi|)
    y = kb.kan_dense_layer_forward(to_dev(tail), to_dev(x)).cpu().numpy()
    rep = ko.error_report(y[rows], ko.dense_layer_forward(tail, x[rows]))
    assert np.isfinite(y).all() and rep["headline"] <= TOL_FP32, rep


def test_fp32_operands_have_no_fp16_range(kb):
    """Up to 16 samples the operands stay fp32: coefficients beyond fp16's range on either side."""
    rng = np.random.default_rng(5)
    coef = (rng.standard_normal((40, 24, 10)) * 10.0 ** rng.uniform(-9, 9, (1, 24, 1))).astype(np.float32)
    x = synth.make_x(6, 16, 40)
    y = kb.kan_dense_layer_forward(to_dev(coef), to_dev(x)).cpu().numpy()
    y_ref, A = ko.dense_layer_forward(coef, x, return_abs=True)
    assert np.all(np.abs(y - y_ref) <= TOL_FP32 * A)


@pytest.mark.parametrize("B", [1, 16])
def test_fp32_operands_hold_weights_rounded_once(kb, B):
    """Up to 16 samples every weight is the fp64 value rounded once to fp32.  One input, output m with the m-th unit
    grid: the outputs are the ten basis values of the sample themselves (a one times a weight and zeros, exact in
    fp32), so they lie within half a unit in the last place (2^-24 of the value) of the oracle's (whose own knots are good to 1e-16)."""
    x = np.random.default_rng(77 + B).uniform(-1.0, 1.0, (400 * B, 1)).astype(np.float32)
    x[:4 * B, 0] = np.linspace(-1.0, 1.0, 4 * B, dtype=np.float32)
    coef = np.eye(10, dtype=np.float32)[None]
    y_ref = ko.dense_layer_forward(coef, x)
    for b in range(0, x.shape[0], B):
        y = kb.kan_dense_layer_forward(to_dev(coef), to_dev(x[b:b + B])).cpu().numpy()
        ref = y_ref[b:b + B]
        assert np.all(np.abs(y - ref) <= 2.0 ** -24 * 1.0001 * np.abs(ref) + 1e-15), np.abs(y - ref).max()

"""The two ways the bucket kernel adds its segments: blocks of up to 17 passes of 512 edges (one strip of running sums
per pass) and larger ones (a run of passes per wave), against the float64 oracle with the bound of the other fp32 kernels."""
import dataclasses

import numpy as np
import pytest

from oracle import kan_oracle as ko
from paper_2512_15742_amd import synth

from kan_testlib import TOL_FP32, gpu_layers, to_dev

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def _forward(P, x):
    from paper_2512_15742_amd import binding as kb
    (L,) = [L.prepare() for L in gpu_layers([P])]
    L.use_prepared(True)
    L.keep_on_bucket_kernel(True)
    assert kb.kan_vq_planned_kernel(L, len(x), 1, kb.KAN_PATH_GATHER) == "kan_bucket"
    first, again = (kb.kan_vq_head_forward([[L]], to_dev(x), path=kb.KAN_PATH_GATHER)[0].cpu().numpy() for _ in range(2))
    assert np.array_equal(first, again, equal_nan=True)              # whatever the waves' timing
    return first


# One bucket and batch 4: 64 blocks per sample, so a block holds n_in * n_out / 64 edges, rounded to whole outputs.
@pytest.mark.parametrize("n_in,n_out", [
    (512, 1024),       # 8192 edges: 16 passes exactly
    (513, 1024),       # 8208 from unaligned starts: the 17th pass
    (512, 1088),       # 8704: 17 passes exactly
    (515, 1088),       # 8755: runs of one and two passes
    (4096, 150),       # segments of 8 passes: over several whole runs
    (16, 40000),       # 625 short segments per block
    (3, 200000),       # 1024 outputs per block, the most there are: runs of hundreds of segments
])
@pytest.mark.parametrize("cb,gb", [("i8", "f16"), ("f32", "f32")])
@pytest.mark.parametrize("skew", [False, True])
def test_segments_of_a_block(n_in, n_out, cb, gb, skew):
    rows = (8192 if cb == "i8" else 2048) // (2 if n_in > 2048 else 1)
    P = synth.make_layer(n_in + n_out, n_in, n_out, 3 * rows if skew else rows, cb_dtype=cb, gb_dtype=gb)
    if skew:           # outputs that own whole stretches of a bucket, and as many that have no edge in it
        third = n_out // 3
        P.idx[:, :third] %= rows
        P.idx[:, 2 * third:] = P.idx[:, 2 * third:] % rows + 2 * rows
    x = synth.make_x(9, 4, n_in)
    y_ref, A = ko.vq_layer_forward(x, **P.as_dict(), return_abs=True)
    rep = ko.error_report(_forward(P, x), y_ref, A)
    assert rep["headline"] <= TOL_FP32 and rep["strict"] <= TOL_FP32, rep


# Batch 4, 64 blocks per sample: up to 17 passes (8704 edges) a block in the first line, runs of passes in the second.
@pytest.mark.parametrize("n_in,n_out,K", [
    (600, 512, 2000), (1033, 300, 2000), (64, 4096, 2000), (700, 640, 60000),
    (1033, 1100, 2000), (600, 2000, 2000), (24, 40000, 2000), (2100, 1300, 60000)])
@pytest.mark.parametrize("cb,gb", [("i8", "f16"), ("f32", "f32")])
def test_outputs_of_unequal_scale_keep_their_own_error(n_in, n_out, K, cb, gb):
    """An output's error is in proportion to its own terms, whatever the scale of the outputs beside it: every one
    within 1e-5 of the sum of its terms' magnitudes, next to outputs of 1,000 times that."""
    P = synth.make_layer(n_in + 2 * n_out, n_in, n_out, K, cb_dtype=cb, gb_dtype=gb)
    scale = np.where(np.arange(n_out) % 2 == 0, 1.0, 1000.0).astype(np.float32)
    gain = (P.gain.astype(np.float32) * scale).astype(P.gain.dtype)
    bias = np.zeros_like(P.bias)
    P = dataclasses.replace(P, gain=gain, bias=bias)
    x = synth.make_x(11, 4, n_in)
    y_ref, A = ko.vq_layer_forward(x, **P.as_dict(), return_abs=True)
    rep = ko.error_report(_forward(P, x), y_ref, A)
    assert rep["strict"] <= TOL_FP32, rep


@pytest.mark.parametrize("n_in,n_out", [(600, 512), (24, 4096), (1033, 1100), (24, 40000)])
def test_products_near_the_largest_number_stay_with_their_outputs(n_in, n_out):
    """Every fourth output's sum passes the range of fp32 from finite products; the others must not notice."""
    P = synth.make_layer(n_in + 3 * n_out, n_in, n_out, 2000, cb_dtype="f32", gb_dtype="f32")
    big = np.arange(n_out) % 4 == 1
    gain = P.gain.copy()
    gain[:, big] = 3e38
    P = dataclasses.replace(P, gain=gain)
    x = synth.make_x(12, 4, n_in)
    y = _forward(P, x)
    y_ref, A = ko.vq_layer_forward(x, **P.as_dict(), return_abs=True)
    rep = ko.error_report(y[:, ~big], y_ref[:, ~big], A[:, ~big])
    assert np.isfinite(y[:, ~big]).all() and rep["strict"] <= TOL_FP32, rep


@pytest.mark.parametrize("n_in,n_out", [(513, 1024), (600, 1200)])
def test_a_non_finite_codeword_stays_with_its_outputs(n_in, n_out):
    P = synth.make_layer(3, n_in, n_out, 2048, cb_dtype="f32", gb_dtype="f32")
    P.idx[P.idx == 7] = 8
    hit = np.zeros(n_out, dtype=bool)
    hit[[0, n_out // 2, n_out - 1]] = True
    P.idx[[[0], [n_in // 2], [n_in - 1]], np.flatnonzero(hit)] = 7
    cb = P.codebook.copy()
    cb[7] = np.inf
    x = synth.make_x(4, 4, n_in)
    y = _forward(dataclasses.replace(P, codebook=cb), x)
    y_ref = ko.vq_layer_forward(x, **P.as_dict())
    assert not np.isfinite(y[:, hit]).any()
    assert ko.error_report(y[:, ~hit], y_ref[:, ~hit])["headline"] <= TOL_FP32

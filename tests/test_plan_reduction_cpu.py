"""Layers whose partial sums only a reduction launch would add stay whole where that launch costs more than the cut saves
(a call of one layer needs a workspace only for partial sums): host logic, no GPU."""
import pytest

from paper_2512_15742_amd import binding as kb

from test_abi_cpu import _head_ws

I8 = dict(gb_dtype=kb.KAN_F16, cb_dtype=kb.KAN_I8)


@pytest.mark.parametrize("n_in", [17, 24, 31, 32])
@pytest.mark.parametrize("B", [2, 16, 31])
@pytest.mark.parametrize("n_out,heads", [(8, 1), (333, 1), (1024, 1), (128, 6)])
def test_last_layers_of_two_steps_are_one_launch(n_in, B, n_out, heads):
    assert _head_ws(kb.lib(), (n_in, n_out), heads, B, kb.KAN_PATH_GATHER, **I8) == 0


@pytest.mark.parametrize("path,n_in,n_out,heads,B", [
    (kb.KAN_PATH_GATHER, 82, 2736, 19, 24), (kb.KAN_PATH_GATHER, 34, 387, 13, 16), (kb.KAN_PATH_GATHER, 31, 3724, 7, 48),
    (kb.KAN_PATH_GATHER, 21, 303, 39, 54), (kb.KAN_PATH_MFMA, 24, 128, 1, 16), (kb.KAN_PATH_MFMA, 31, 327, 35, 30),
    (kb.KAN_PATH_MFMA, 30, 3297, 8, 10), (kb.KAN_PATH_MFMA, 147, 866, 46, 36)])
def test_cuts_that_cost_more_than_they_save_are_not_made(path, n_in, n_out, heads, B):
    assert _head_ws(kb.lib(), (n_in, n_out), heads, B, path, **I8) == 0


def test_cuts_that_pay_for_their_reduction_are_made():
    for path, n_in, n_out, B in ((kb.KAN_PATH_GATHER, 64, 32, 16), (kb.KAN_PATH_GATHER, 48, 128, 31),
                                 (kb.KAN_PATH_GATHER, 24, 128, 37), (kb.KAN_PATH_MFMA, 64, 128, 16)):
        assert _head_ws(kb.lib(), (n_in, n_out), 1, B, path, **I8) > 0


def test_a_middle_layer_whose_slices_the_next_one_does_not_take():
    """333 inputs are not taken as slices (rows of fours): the layer in front of them is whole, and the call's workspace
    is the two hidden buffers and the last layer's sums."""
    L, hidden = kb.lib(), (16 * 333 * 4 + 255) // 256 * 256
    last = _head_ws(L, (333, 21), 1, 16, kb.KAN_PATH_GATHER, **I8)
    assert _head_ws(L, (32, 333, 21), 1, 16, kb.KAN_PATH_GATHER, **I8) == 2 * hidden + last
